// State pass for the maps 128 -> 256 -> 256 (the paper's default widths): phi_k on the linear tokens and the partial tiles of
// S = sum phi_k(k_j)^T v_j (256 x 128) and z = sum phi_k(k_j), per chunk of tokens, for state_reduce_kernel.  gfx950 only.
//
// Two roles per workgroup, as in the state pass of the narrow maps (ha_state.hip), two waves per SIMD:
//   * waves 0 - 3 evaluate phi_k (ha_mlp256.h), 32 token rows each, one hidden block per step from a 24 KiB slab of weights;
//   * waves 4 - 7 own two 32-row blocks of [S | z] each (160 accumulator registers).  They stream the slabs into a double
//     buffer (all of W1 and W2 is 192 KiB per head: it does not fit), fetch the V rows, and contract the previous tile, 16 of
//     its 128 tokens per step, both operands through transposing LDS reads.
// A barrier opens every step (slab in place, the other one free); one more, after the eight steps and the output stage, lets
// phi and V of the tile replace those of the previous one, and the next step's barrier publishes them.
// Every wave passes the same barriers: nine per tile and one at the end.
//
// Bound: matrix cores, 400 instructions of 32 cycles per SIMD and 128-token tile (12.8 k cycles), next to 5 k cycles of
// exponentials and packing that nothing covers.  The next hidden block is formed under the products of the current one (so a slab
// brings the rows of W1 of the block after its own).  Measured in traces of 60 forwards, one box, with the next block as a chain at the
// head of its own step / here: 480p / 81 frames, 12 heads, R = 4  143 / 130 us; B = 2, N = 5003, R = 3, fp32  61 / 59 us.  (One role with
// the weights staged per tile in two rounds had taken 222 and 108 where the first form with two roles took 128 and 66.)
#include "ha_mlp256.h"
#include "ha_plan.h"

namespace ha {

template <bool F32, bool ACT0, bool P2>
__global__ __launch_bounds__(512, 1) void state256_kernel(const void *__restrict__ k, const void *__restrict__ v,
                                                          const bf16x8 *w1f_all, const bf16x8 *w2f_all,
                                                          const float *__restrict__ b1_all, const float *__restrict__ b2_all,
                                                          float *__restrict__ part, int H, int NL, int R, int G, int CH, int P,
                                                          int act, int64_t sb, int64_t sh, int64_t sn, int N, int CC, int nsub) {
  constexpr int D = 128, HD = 256, F = 256, TOK = 128, KS = D / 16, HB = HD / 32, FB = F / 32, NCB = D / 32 + 1, NT = FB * NCB;
  constexpr int SLAB = kSlabChunks * 64;
  typedef RowTile<D> RT;
  constexpr int VROW = RT::ROWB, PROW = 2 * F, PPR = RT::PPR;
  __shared__ bf16x8 slab[2][SLAB];
  __shared__ __align__(16) char phi_t[TOK * PROW];
  __shared__ __align__(16) char v_t[TOK * VROW];
  __shared__ __align__(16) float blds[HD + F];

  const int chunk = blockIdx.x, bh = blockIdx.y, h = bh % H;
  const int64_t base = (int64_t)(bh / H) * sb + (int64_t)h * sh;
  const int tid = threadIdx.x, lane = tid & 63, r = lane & 31, g = lane >> 5;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int w = wave & 3;                              // index within the role
  const bf16x8 *w1g = w1f_all + (int64_t)h * (HD * D / 8), *w2g = w2f_all + (int64_t)h * (F * HD / 8);
  // (requested ahead of everything, written to LDS behind the request of the first K rows: B = 2, N = 5003, fp32 3 % of this kernel)
  float bias1 = 0.f, bias2 = 0.f;
  static_assert(HD == 256 && F == 256, "the first four waves write them");
  if (tid < 256) {
    if (b1_all) bias1 = b1_all[(int64_t)h * HD + tid];
    if (b2_all) bias2 = b2_all[(int64_t)h * F + tid];
  }
  const LinearMap lmap(R, G);

  // this workgroup's range of linear tokens: chunk number `chunk` of CH tokens, or (chunk-causal variant) piece
  // chunk % nsub of the linear tokens of causal chunk chunk / nsub
  int lt_begin = chunk * CH;
  int lt_end = min(lt_begin + CH, NL);
  if (CC > 0) {
    const int cc = chunk / nsub, lo = cc * CC, hi = min(lo + CC, N);
    lt_begin = lo - softmax_before(lo, R, G) + (chunk % nsub) * CH;
    lt_end = min(lt_begin + CH, hi - softmax_before(hi, R, G));
  }

  // phi tile: row-major, 512 bytes per token; 16-byte piece p of row t sits at p ^ psw(t), psw(t) = 4 (t % 4) + (t / 4) % 4:
  // the 32 rows one write instruction touches fall on 16 different pieces, and a transposing read finds its four rows in
  // four different 64-byte groups
  if (wave < 4) {
    // =============================== the feature map: phi_k of 32 token rows per wave ===============================
    const float *b1 = &blds[0], *b2 = &blds[HD];
    const int tf = w * 32 + r;
    auto load_k = [&](int t0, bf16x8 (&dst)[KS]) {
      const int tok = lmap.token(min(t0 + tf, NL - 1));   // rows past the end repeat the last linear token; masked later
#pragma unroll
      for (int ks = 0; ks < KS; ++ks) dst[ks] = load8<F32>(k, base + (int64_t)tok * sn + 16 * ks + 8 * g);
    };
    bf16x8 xf[KS];
    load_k(lt_begin, xf);
    blds[tid] = bias1;
    blds[HD + tid] = bias2;
    const lds_frag_ptr sl0 = (lds_frag_ptr)&slab[0][0], sl1 = (lds_frag_ptr)&slab[1][0];
    u32x4 h_hi[2], h_lo[2];                            // the hidden block of the current step
    f32x16 hh;
    auto first_block = [&]() {                         // hidden block 0 of the tile in xf: its rows of W1 are with slab 7
      bf16x8 wl[KS];
#pragma unroll
      for (int ks = 0; ks < KS; ++ks) wl[ks] = frag_at(sl1, ks, lane);
      hh = column_tile(b1, 0, g);
#pragma unroll
      for (int ks = 0; ks < KS; ++ks) hh = mfma32(wl[ks], xf[ks], hh);
    };
    auto first_split = [&]() {
#pragma unroll
      for (int x = 0; x < 16; x += 2) split2(hh, x, h_hi, h_lo);
    };
    __syncthreads();                                   // the biases and W1 of block 0 are in LDS
    if (lt_begin < lt_end) {
      first_block();
      first_split();
    }
    for (int t0 = lt_begin; t0 < lt_end; t0 += TOK) {
      f32x16 u[FB];
#pragma unroll
      for (int fb = 0; fb < FB; ++fb) u[fb] = column_tile(b2, fb, g);
      bf16x8 fr[2][2];
#pragma unroll 1
      for (int hb = 0; hb + 1 < HB; ++hb) {
        __syncthreads();                               // slab hb is in place
        const lds_frag_ptr sl = (hb & 1) ? sl1 : sl0;
        read_group256(sl + KS * 64, 0, lane, fr);
        hidden_block_products<true>(sl + KS * 64, sl, b1, hb + 1, xf, lane, g, fr, h_hi, h_lo, u);
      }
      load_k(t0 + TOK, xf);                            // the next tile's rows travel under the last step and the output stage
      __syncthreads();                                 // slab 7 is in place
      read_group256(sl1 + KS * 64, 0, lane, fr);
      hidden_block_products<false>(sl1 + KS * 64, nullptr, nullptr, 0, xf, lane, g, fr, h_hi, h_lo, u);
      phi256_output<ACT0, P2>(u, act, P);
      first_block();                                   // of the next tile: its products run under the packing below
      if (t0 + TOK > lt_end) {                         // ragged end of the range: padded tokens add nothing
        // (by selection: a padded row may be a token of the next causal chunk, whose features need not be finite)
        const bool keep = t0 + tf < lt_end;
#pragma unroll
        for (int fb = 0; fb < FB; ++fb)
#pragma unroll
          for (int x = 0; x < 16; ++x) u[fb][x] = keep ? u[fb][x] : 0.f;
      }
      // registers 4 q .. 4 q + 3 of tile fb are channels 32 fb + 8 q + 4 g .. + 3: half of 16-byte piece 4 fb + q
      typedef unsigned u32x2 __attribute__((ext_vector_type(2)));
      u32x2 four[FB][4];
#pragma unroll
      for (int fb = 0; fb < FB; ++fb)
#pragma unroll
        for (int q = 0; q < 4; ++q)
          four[fb][q] = u32x2{pack_bf16(u[fb][4 * q], u[fb][4 * q + 1]), pack_bf16(u[fb][4 * q + 2], u[fb][4 * q + 3])};
      int row = tf;
      asm volatile("" : "+v"(row));                    // the addresses below are formed here, not kept across the tile
      const int psw = 4 * (row & 3) + ((row >> 2) & 3), at = row * PROW + 8 * g;
      __syncthreads();                                 // the contraction of the previous tile has read phi_t
#pragma unroll
      for (int fb = 0; fb < FB; ++fb)
#pragma unroll
        for (int q = 0; q < 4; ++q) *reinterpret_cast<u32x2 *>(phi_t + at + (((4 * fb + q) ^ psw) << 4)) = four[fb][q];
      first_split();
    }
    __syncthreads();                                   // the last tile is in place
    return;
  }

  // ========================= the weights, V, and the contraction over the tokens (waves 4 .. 7) =========================
  f32x16 acc[2][NCB];                                  // row blocks 2 w, 2 w + 1 of [S | z]
#pragma unroll
  for (int e = 0; e < 2; ++e)
#pragma unroll
    for (int i = 0; i < NCB; ++i)
#pragma unroll
      for (int x = 0; x < 16; ++x) acc[e][i][x] = 0.f;
  const unsigned lane_off = lane * 16;
  // Slab hb into buffer hb % 2, six chunks per wave: the columns of W2 of hidden block hb, in front of them the rows of W1 of the
  // block after it (behind the last one: of block 0, for the next tile), which is formed under this one's products.
  auto dma = [&](const bf16x8 *gp, bf16x8 *to) {
    const unsigned l = __builtin_amdgcn_readfirstlane((unsigned)(uintptr_t)(__attribute__((address_space(3))) void *)to);
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2" ::"s"(l), "v"(lane_off), "s"(gp) : "memory");
  };
  auto request = [&](int hb) {
#pragma unroll
    for (int i = 0; i < kSlabChunks / 4; ++i) {
      const int c = 4 * i + w;
      dma(slab_chunk(w1g, w2g, i < 2 ? (hb + 1) % HB : hb, c), &slab[hb & 1][c * 64]);
    }
  };
#pragma unroll
  for (int i = 0; i < 2; ++i) dma(slab_chunk(w1g, w2g, 0, 4 * i + w), &slab[1][(4 * i + w) * 64]);   // W1 of block 0 for the first tile
  request(0);
  // transposing reads: lane = (group tm, row ti, columns ta); see ds_read_tr
  const int tm = lane >> 4, ti = (lane >> 2) & 3, ta = lane & 3, tg = tm >> 1;
  int v_base[D / 32], a_base[2][2];
#pragma unroll
  for (int cb = 0; cb < D / 32; ++cb)
    v_base[cb] = (8 * tg + ti) * VROW + (((4 * cb + 2 * (tm & 1) + (ta >> 1)) ^ RT::sw(ti)) << 4) + 8 * (ta & 1);
#pragma unroll
  for (int e = 0; e < 2; ++e)
#pragma unroll
    for (int jj = 0; jj < 2; ++jj)
      a_base[e][jj] = (8 * tg + ti) * PROW +
                      (((4 * (2 * w + e) + 2 * (tm & 1) + (ta >> 1)) ^ (4 * ti + ((2 * tg + jj) & 3))) << 4) + 8 * (ta & 1);
  // V rows: global -> registers, then into v_t (row-major, four rows per instruction).  This lane's rows are 4 RPI apart: one exact division gives the first one's group, the others follow by adding the
  // quotient and remainder of the row distance (a tile that reaches past the last linear token clamps every row).
  constexpr int RPI = 1024 / VROW, NVI = TOK / RPI;
  const int v_row = lane / PPR, v_pp = lane % PPR;
  const int step_q = (4 * RPI) / lmap.d, step_r = (4 * RPI) % lmap.d;
  bf16x8 vreg[NVI / 4];
  auto load_v = [&](int t0) {
    const bool whole = t0 + TOK <= NL;                 // wave-uniform
    const int i0 = t0 + w * RPI + v_row;
    int grp = 0, rem = 0;
    if (whole && lmap.g != 0) {
      grp = lmap.token(i0) - i0;                       // (i0 / d + 1) g
      rem = i0 - (grp / lmap.g - 1) * lmap.d;
    }
#pragma unroll
    for (int c = 0; c < NVI / 4; ++c) {
      const int row = (4 * c + w) * RPI + v_row;
      int tok;
      if (whole) {
        tok = t0 + row + grp;
        rem += step_r;
        const bool carry = rem >= lmap.d;
        rem -= carry ? lmap.d : 0;
        grp += (step_q + (carry ? 1 : 0)) * lmap.g;
      } else {
        tok = lmap.token(min(t0 + row, NL - 1));
      }
      vreg[c] = load8<F32>(v, base + (int64_t)tok * sn + (v_pp ^ RT::sw(row)) * 8);
    }
  };
  const __bf16 one = static_cast<__bf16>(r == 0 ? 1.0f : 0.0f);     // the "1" column that yields z
  const bf16x8 ones = bf16x8{one, one, one, one, one, one, one, one};
  auto contract = [&](int ks) {                        // 16 tokens of the tile in phi_t, v_t
    bf16x8 a8[2], b8[D / 32];
#pragma unroll
    for (int e = 0; e < 2; ++e)
      a8[e] = join(ds_read_tr(phi_t, a_base[e][0] + ks * 16 * PROW), ds_read_tr(phi_t, a_base[e][1] + (ks * 16 + 4) * PROW));
#pragma unroll
    for (int cb = 0; cb < D / 32; ++cb)
      b8[cb] = join(ds_read_tr(v_t, v_base[cb] + ks * 16 * VROW), ds_read_tr(v_t, v_base[cb] + (ks * 16 + 4) * VROW));
#pragma unroll
    for (int cb = 0; cb < NCB; ++cb)
#pragma unroll
      for (int e = 0; e < 2; ++e) acc[e][cb] = mfma32(a8[e], cb < D / 32 ? b8[cb] : ones, acc[e][cb]);
  };
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  __syncthreads();                                     // the biases and W1 of block 0 are in LDS
  for (int t0 = lt_begin; t0 < lt_end; t0 += TOK) {
#pragma unroll 1
    for (int hb = 0; hb < HB; ++hb) {
      asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); // slab hb was requested a step ago
      __syncthreads();                                 // slab hb is in place, its predecessor has been read
      if (hb + 1 < HB) request(hb + 1);
      else if (t0 + TOK < lt_end) request(0);
      if (t0 > lt_begin) contract(hb);
    }
    load_v(t0);                                        // travels while the other waves are in the output stage
    __syncthreads();                                   // the previous tile has been contracted
#pragma unroll
    for (int c = 0; c < NVI / 4; ++c)
      *reinterpret_cast<bf16x8 *>(v_t + ((4 * c + w) * RPI + v_row) * VROW + (v_pp << 4)) = vreg[c];
  }
  __syncthreads();                                     // the last tile is in place
  if (lt_begin < lt_end)
#pragma unroll
    for (int ks = 0; ks < TOK / 16; ++ks) contract(ks);
  float *dst = part + (((int64_t)bh * gridDim.x + chunk) * NT + (int64_t)w * 2 * NCB) * 1024;
#pragma unroll
  for (int e = 0; e < 2; ++e)
#pragma unroll
    for (int i = 0; i < NCB; ++i)
#pragma unroll
      for (int x = 0; x < 16; ++x) dst[(e * NCB + i) * 1024 + x * 64 + lane] = acc[e][i][x];
}

hipError_t launch_state256(const Plan &pl, const void *k, const void *v, const ha_feature_map &fm, void *ws, hipStream_t st) {
  dim3 grid(pl.n_chunks, pl.B * pl.H);
  char *wsb = static_cast<char *>(ws);
  const bf16x8 *w1f = reinterpret_cast<bf16x8 *>(wsb + pl.off_w1k), *w2f = reinterpret_cast<bf16x8 *>(wsb + pl.off_w2k);
  float *part = reinterpret_cast<float *>(wsb + pl.off_part);
#define HA_STATE256(F32, ACT0, P2) \
  state256_kernel<F32, ACT0, P2><<<grid, 512, 0, st>>>(k, v, w1f, w2f, fm.b1, fm.b2, part, pl.H, pl.NL, pl.R, pl.G, pl.CH, pl.P, \
                                                       pl.act_k, pl.sb, pl.sh, pl.sn, pl.N, pl.CC, pl.nsub)
#define HA_STATE256_MAP(F32) \
  do { \
    if (pl.act_k != HA_ACT_SOFTMAX) HA_STATE256(F32, false, false); \
    else if (pl.P == 2) HA_STATE256(F32, true, true); \
    else HA_STATE256(F32, true, false); \
  } while (0)
  if (pl.f32) HA_STATE256_MAP(true); else HA_STATE256_MAP(false);
#undef HA_STATE256_MAP
#undef HA_STATE256
  return hipGetLastError();
}

}  // namespace ha
