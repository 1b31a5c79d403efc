// Feature maps of any width (Attention Surgery, Sec. 3.2 "Characterization of phi"; Tab. "phi": d -> P d -> P d
// for P = 2, 3, 4 and the three-layer P = 6 map), gfx950.  The fused kernels keep a token's hidden activations and
// all its output channels in registers, which ends at 256 channels.  Here every layer is a pass of its own and
// activations travel through HBM, in exactly the register image the next product wants:
//
//   wide_prep_kernel       weight matrices -> A-operand fragments (natural order for layer 1, chained after it)
//   (ha_wide_mlp.hip)      h^T = relu(W1 x^T + b1) on the way into  h'^T = relu(W h^T + b)  or  u^T = W h^T + b  (last
//                          layer: fp32 pre-activations); h' as hi + lo bf16
//   (output stage)         softmax / exp / relu over all channels of a token, slice powers, bf16: applied by the two
//                          consumers below while they read the pre-activations, so phi never visits HBM
//   wide_state_kernel      [S | z] += phi_k^T [V | 1], a slab of 256 or 128 features per workgroup
//   wide_lin_kernel        n_i = phi_q(q_i) S   (fp32, in the layout of the query kernel's accumulators), e_i = phi_q(q_i).z
// The query kernel then adds n_i and e_i in its epilogue instead of evaluating phi_q itself.
//
// Register images ("C image" of a 32-token block tb of (batch, head) bh; lane = 32 g + r owns token 32 tb + r):
//   activations   bf16x8 [bh][tb][W/32][2][64]   piece (block c, half s) = channels 32 c + crow(8 s + t, g), t = 0..7,
//                                                i.e. the B operand ("chained" order) of the next product
//   fp32 tiles    f32x4  [bh][tb][W/32][4][64]   piece (block c, quad x) = channels 32 c + crow(4 x + j, g), j = 0..3
//   the same for the state pass: lane = 32 g + r owns channel 32 c + r, piece (block c, quad x) = tokens 32 tb + crow(4 x + j, g)
#include "ha_mlp128.h"
#include "ha_plan.h"

namespace ha {

// ------------------------------------------------------------------------------------------------
// wide_prep_kernel: grid (2048 weights each, H).  W [H][NOUT][K] (io dtype) of all layers of a map -> fragments, see weight_piece.
// (A launch per layer takes 5 - 8 us each, one behind the other: three layers at 768, 12 heads, 21 us, in one launch 14; whole calls with two
// layers, H = 2, N = 2000, 384 wide 100.5 -> 97.2, H = 1, N = 300, 768 wide 140.3 -> 136.6.)
struct WidePrepLayer {
  const void *w;
  bf16x8 *frags;
  int NOUT, K, first;                 // first: the layer's first column of the grid
  bool chained;
};
struct WidePrepMap {
  WidePrepLayer layer[3];
};
template <bool F32>
__global__ __launch_bounds__(256) void wide_prep_kernel(WidePrepMap m) {
  const int col = blockIdx.x;
  const WidePrepLayer l = col >= m.layer[2].first ? m.layer[2] : col >= m.layer[1].first ? m.layer[1] : m.layer[0];
  const int piece = (col - l.first) * 256 + threadIdx.x;
  const int64_t n = (int64_t)l.NOUT * l.K, base = blockIdx.y * n;
  if (piece >= n / 8) return;
  l.frags[base / 8 + piece] = l.chained ? weight_piece<F32, true>(l.w, base, l.K, piece) : weight_piece<F32, false>(l.w, base, l.K, piece);
}

// ------------------------------------------------------------------------------------------------
// Output stage of a feature map, applied by the consumers of phi while they read the fp32 pre-activations (so phi
// itself never visits HBM): normalisation (softmax: against the maximum and sum combined from the per-128-channel-block
// values the last layer left behind), slice powers, rounding.
constexpr int WIDE_FMAX = 768;

struct WideOutStage {
  float off, inv, inv_groups;     // softmax: exp2(u log2 e + off) * inv;  1 / (8-channel groups per slice)
  int act;
};

// One lane's view (token 32 tb + lane % 32) of the softmax statistics of its token.
static __device__ __forceinline__ WideOutStage wide_out_stage(const float *__restrict__ stat, int64_t bh_tb, int F, int act,
                                                              int P, int lane) {
  WideOutStage o;
  o.off = 0.f; o.inv = 1.f; o.act = act;
  o.inv_groups = 8.0f * (float)P / (float)F;
  if (act == 0) {
    const int nblk = F / 128;
    const float *st = stat + (bh_tb * nblk * 2) * 64 + lane;
    float m = -INFINITY;
    for (int b = 0; b < nblk; ++b) m = fmaxf(m, st[b * 128]);
    float sum = 0.f;
    for (int b = 0; b < nblk; ++b) sum += st[b * 128 + 64] * fast_exp2((st[b * 128] - m) * kLog2e);
    o.off = -m * kLog2e;
    o.inv = 1.0f / sum;
  }
  return o;
}

// phi of the 32-channel tile fb of one token block from its fp32 C image piece: the two bf16 pieces (chained order)
// the next product takes as its B operand; zero for tokens past the end.
static __device__ __forceinline__ void wide_phi_tile(const f32x4 (&raw)[4], int fb, const WideOutStage &o, bool valid,
                                                     bf16x8 (&out)[2]) {
  f32x16 u;
#pragma unroll
  for (int x4 = 0; x4 < 4; ++x4)
#pragma unroll
    for (int j = 0; j < 4; ++j) u[4 * x4 + j] = raw[x4][j];
  if (o.act == 0) {                                            // one branch per tile, not one per value
#pragma unroll
    for (int v = 0; v < 16; ++v) u[v] = fast_exp2(__builtin_fmaf(u[v], kLog2e, o.off)) * o.inv;
  } else if (o.act == 1) {
#pragma unroll
    for (int v = 0; v < 16; ++v) u[v] = fast_exp2(u[v] * kLog2e);
  } else {
#pragma unroll
    for (int v = 0; v < 16; ++v) u[v] = fmaxf(u[v], 0.f);
  }
#pragma unroll
  for (int s = 0; s < 2; ++s) {
    f32x8 t8;
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      // slice power - 1 = (8-channel group index) / (groups per slice), wave-uniform; exact in fp32 for these sizes
      const int extra = (int)(((float)(4 * fb + 2 * s + i / 4) + 0.5f) * o.inv_groups);
      const float t0 = u[8 * s + i], t2 = t0 * t0;
      float t = (extra & 1) ? t2 : t0;                           // t0^(extra + 1), extra in 0..7
      t = (extra & 2) ? t * t2 : t;
      t = (extra & 4) ? t * (t2 * t2) : t;
      t8[i] = valid ? t : 0.f;
    }
    out[s] = __builtin_convertvector(t8, bf16x8);
  }
}

// ------------------------------------------------------------------------------------------------
// wide_state_kernel: [S | z] += phi_k^T [V | 1] of one chunk of tokens, one (batch, head) and 32 NW features, a 32-row block of them
// per wave.  The pre-activations arrive with a channel per lane and the tokens in the registers (WideMlpLayer::channel_lanes), so
// phi_k, formed as they are read, is the A operand of the contraction as it stands; only the V rows go through LDS (row-major,
// double buffered, 64 tokens at a time, one barrier per 64; transposing reads), and with them what the output stage needs per token.
// Both travel a tile ahead, the pre-activations a tile ahead in registers.  The workgroups of a chunk are consecutive on one XCD,
// so that its V rows leave HBM once.
// Partial tiles go where state_kernel puts them (part[bh][chunk][row block * NCB + column block][v][lane]), so state_reduce_kernel
// serves both.
// Bound: HBM, the fp32 pre-activations.  768 wide, 480p / 81 frames, R = 8, 12 heads (1.06 GB of them): 467 us with phi transposed
// through LDS two bytes at a time by workgroups of 128 features (8 % matrix cores, 67 % of the wave cycles waiting; 465 with V
// fetched once), 512 with the statistics waited for where they are requested, 265 with them ahead, 240 us with the pre-activations
// read non-temporally (ONCE; 4.9 TB/s).
template <int NW, bool F32, bool ONCE>
__global__ __launch_bounds__(64 * NW, 2) void wide_state_kernel(const f32x4 *__restrict__ u_img, const float *__restrict__ stat,
                                                                const void *__restrict__ v, float *__restrict__ part, int H,
                                                                int NL, int R, int G, int CH, int F, int n_tb, int act, int P,
                                                                int64_t sb, int64_t sh, int64_t sn, int n_chunks, int n_pairs) {
  constexpr int D = 128, TOK = 64, NCB = D / 32 + 1;
  typedef RowTile<D> RT;
  constexpr int VROW = RT::ROWB, PPR = RT::PPR, VPT = TOK * PPR / (64 * NW);
  __shared__ __align__(16) char v_t[2][TOK * VROW];
  __shared__ __align__(16) float tok_off[2][TOK], tok_inv[2][TOK];
  const int FB = F / 32, nz = FB / NW;
  const int in_xcd = blockIdx.x >> 3, pair = (in_xcd / nz) * 8 + (blockIdx.x & 7), zb = in_xcd % nz;
  if (pair >= n_pairs) return;
  const int bh = pair / n_chunks, chunk = pair - bh * n_chunks, h = bh % H;
  const int64_t base = (int64_t)(bh / H) * sb + (int64_t)h * sh;
  const int tid = threadIdx.x, lane = tid & 63, r = lane & 31, g = lane >> 5;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6), fb = zb * NW + w;
  const LinearMap lmap(R, G);
  const int lt_begin = chunk * CH, lt_end = min(lt_begin + CH, NL);

  // V rows of a tile and (wave 0) the statistics of its tokens, on their way in registers
  constexpr int MAXB = WIDE_FMAX / 128;
  const int nblk = F / 128;
  bf16x8 vreg[VPT];
  float st_m[MAXB], st_s[MAXB];
  auto load_tile = [&](int t0) {
#pragma unroll
    for (int c = 0; c < VPT; ++c) {
      const int i = c * 64 * NW + tid, row = i / PPR, pp = i % PPR;
      const int tok = lmap.token(min(t0 + row, NL - 1));
      vreg[c] = load8<F32>(v, base + (int64_t)tok * sn + (pp ^ RT::sw(row)) * 8);
    }
    if (act == 0 && w == 0) {
      const int tb = min(t0 / 32 + (lane >> 5), n_tb - 1);
      const float *st = stat + ((int64_t)bh * n_tb + tb) * nblk * 128 + r;
#pragma unroll
      for (int b = 0; b < MAXB; ++b) {                 // (blocks there are not repeat the first)
        st_m[b] = st[(b < nblk ? b : 0) * 128];
        st_s[b] = st[(b < nblk ? b : 0) * 128 + 64];
      }
    }
  };
  // (fragment 32-token block tb, quad x4): tokens crow(4 x4 + j, g) of channel 32 fb + r
  f32x4 raw[2][4];
  auto load_u = [&](int t0, int blk) {
    const f32x4 *src = u_img + (((int64_t)bh * n_tb + min(t0 / 32 + blk, n_tb - 1)) * FB + fb) * 256 + lane;
#pragma unroll
    for (int x4 = 0; x4 < 4; ++x4) raw[blk][x4] = ONCE ? __builtin_nontemporal_load(&src[x4 * 64]) : src[x4 * 64];
  };
  f32x16 acc[NCB];
#pragma unroll
  for (int i = 0; i < NCB; ++i)
#pragma unroll
    for (int x = 0; x < 16; ++x) acc[i][x] = 0.f;
  // slice power - 1 of this lane's channel = (8-channel group) / (groups per slice); exact in fp32 for these sizes
  const int extra = (int)(((float)(4 * fb + (r >> 3)) + 0.5f) * (8.0f * (float)P / (float)F));
  // transposing reads: lane = (group tm, row ti, columns ta); slot (g, t) of half s holds token 16 s + crow(t, g) (see ds_read_tr)
  const int tm = lane >> 4, ti = (lane >> 2) & 3, ta = lane & 3, tg = tm >> 1;
  int v_base[D / 32];
#pragma unroll
  for (int cb = 0; cb < D / 32; ++cb)
    v_base[cb] = (4 * tg + ti) * VROW + (((4 * cb + 2 * (tm & 1) + (ta >> 1)) ^ RT::sw(ti)) << 4) + 8 * (ta & 1);
  const __bf16 one = static_cast<__bf16>(r == 0 ? 1.0f : 0.0f);     // the "1" column that yields z
  const bf16x8 ones = bf16x8{one, one, one, one, one, one, one, one};

  load_tile(lt_begin);
  HA_FENCE();                                          // (in the loop's order: the compiler counts what may be in flight over both ways in)
  load_u(lt_begin, 0);
  HA_FENCE();
  load_u(lt_begin, 1);
  int buf = 0;
  for (int t0 = lt_begin; t0 < lt_end; t0 += TOK, buf ^= 1) {
    // (this buffer was last read two tiles ago: every wave has passed the barrier of the tile between since)
#pragma unroll
    for (int c = 0; c < VPT; ++c) {
      const int i = c * 64 * NW + tid;
      *reinterpret_cast<bf16x8 *>(&v_t[buf][i * 16]) = vreg[c];
    }
    if (act == 0 && w == 0) {
      float m = st_m[0], sum = 0.f;
#pragma unroll
      for (int b = 1; b < MAXB; ++b) m = fmaxf(m, st_m[b]);
#pragma unroll
      for (int b = 0; b < MAXB; ++b) sum += b < nblk ? st_s[b] * fast_exp2((st_m[b] - m) * kLog2e) : 0.f;
      tok_off[buf][lane] = -m * kLog2e;
      tok_inv[buf][lane] = 1.0f / sum;
    }
    __syncthreads();
    const int t1 = t0 + TOK < lt_end ? t0 + TOK : t0;
    load_tile(t1);
    HA_FENCE();
#pragma unroll
    for (int blk = 0; blk < 2; ++blk) {
      f32x16 u;
#pragma unroll
      for (int x4 = 0; x4 < 4; ++x4)
#pragma unroll
        for (int j = 0; j < 4; ++j) u[4 * x4 + j] = raw[blk][x4][j];
      load_u(t1, blk);
      if (act == 0) {                                            // one branch per block, not one per value
#pragma unroll
        for (int x4 = 0; x4 < 4; ++x4) {
          const f32x4 o4 = *reinterpret_cast<const f32x4 *>(&tok_off[buf][32 * blk + 8 * x4 + 4 * g]);
          const f32x4 i4 = *reinterpret_cast<const f32x4 *>(&tok_inv[buf][32 * blk + 8 * x4 + 4 * g]);
#pragma unroll
          for (int j = 0; j < 4; ++j) u[4 * x4 + j] = fast_exp2(__builtin_fmaf(u[4 * x4 + j], kLog2e, o4[j])) * i4[j];
        }
      } else if (act == 1) {
#pragma unroll
        for (int x = 0; x < 16; ++x) u[x] = fast_exp2(u[x] * kLog2e);
      } else {
#pragma unroll
        for (int x = 0; x < 16; ++x) u[x] = fmaxf(u[x], 0.f);
      }
      if (P > 1) {
#pragma unroll
        for (int x = 0; x < 16; ++x) {
          const float a0 = u[x], a2 = a0 * a0;
          float t = (extra & 1) ? a2 : a0;                       // a0^(extra + 1), extra in 0..7
          t = (extra & 2) ? t * a2 : t;
          u[x] = (extra & 4) ? t * (a2 * a2) : t;
        }
      }
      if (t0 + 32 * (blk + 1) > lt_end) {                        // padded tokens of a ragged tile add nothing, whatever they hold
#pragma unroll
        for (int x = 0; x < 16; ++x) u[x] = t0 + 32 * blk + crow(x, g) < lt_end ? u[x] : 0.f;
      }
#pragma unroll
      for (int s = 0; s < 2; ++s) {
        f32x8 t8;
#pragma unroll
        for (int i = 0; i < 8; ++i) t8[i] = u[8 * s + i];
        const bf16x8 phi = __builtin_convertvector(t8, bf16x8);
        const char *vt = &v_t[buf][(32 * blk + 16 * s) * VROW];
#pragma unroll
        for (int cb = 0; cb < D / 32; ++cb)
          acc[cb] = mfma32(phi, join(ds_read_tr(vt, v_base[cb]), ds_read_tr(vt, v_base[cb] + 8 * VROW)), acc[cb]);
        acc[D / 32] = mfma32(phi, ones, acc[D / 32]);
      }
    }
  }
  float *dst = part + ((int64_t)pair * FB + fb) * NCB * 1024;
#pragma unroll
  for (int i = 0; i < NCB; ++i)
#pragma unroll
    for (int x = 0; x < 16; ++x) dst[i * 1024 + x * 64 + lane] = acc[i][x];
}

// ------------------------------------------------------------------------------------------------
// wide_lin_kernel: grid (ceil(n_tb / 8), B*H), 8 waves.  Output stage of phi_q and the linear part of
// Eq. "hybrid" per 32-query block: n^T = S^T phi_q^T (A operand = S^T as hi + lo fragments in chained order,
// state_reduce_kernel's layout; B operand = phi_q, formed tile by tile from the fp32 pre-activations) and e = phi_q . z
// with the rounded phi_q, as the numerator uses it.  Output: n as an fp32 C image of width D, i.e. the layout of the query
// kernel's accumulators; e[bh][token].
// The 16 fragments of S a 32-channel tile meets are the same for all waves: a slab of an LDS ring, one barrier per tile
// (every wave reading its own from L2, 4.7 GB of them: 460 us at 480p / 81 frames, 768 wide, 12 heads; 363 so, and 354 with
// the pre-activations read non-temporally, ONCE).  The
// wave's own tile of pre-activations comes with it, two tiles ahead: the bound is HBM, 1.2 GB of them, and 64 KiB per CU
// are on their way.
// All loads of the loop are LDS-DMA so that the counts below are the only waits.
template <int D, bool ONCE>
__global__ __launch_bounds__(512, 2) void wide_lin_kernel(const f32x4 *u_img, const float *stat, const bf16x8 *st_hi,
                                                          const bf16x8 *st_lo, const float *z, f32x4 *lin, float *e_out, int F,
                                                          int n_tok, int n_tb, int act, int P) {
  constexpr int RB = D / 32, NBUF = 3, SLOT = RB * 4 * 64;
  static_assert(RB * 4 == 16, "two chunks of a slab per wave: the wait below counts them");
  __shared__ bf16x8 ring[NBUF * SLOT];
  __shared__ f32x4 tile[NBUF * 8 * 4 * 64];             // [slot][wave][piece]
  __shared__ __align__(16) float zl[WIDE_FMAX];
  const int bh = blockIdx.y;
  for (int i = threadIdx.x; i < F; i += 512) zl[i] = z[(int64_t)bh * F + i];
  const int lane = threadIdx.x & 63, r = lane & 31, g = lane >> 5;
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const bool live = blockIdx.x * 8 + w < n_tb;          // idle waves keep staging and synchronising
  const int tb = live ? blockIdx.x * 8 + w : n_tb - 1;
  const int FB = F / 32;
  const bool valid = 32 * tb + r < n_tok;
  const unsigned lane_off = lane * 16;
  const f32x4 *usrc = u_img + ((int64_t)bh * n_tb + tb) * FB * 256;
  auto dma = [&](const void *to, const void *from) {
    const unsigned l = __builtin_amdgcn_readfirstlane((unsigned)(uintptr_t)(__attribute__((address_space(3))) void *)to);
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2" ::"s"(l), "v"(lane_off), "s"(from) : "memory");
  };
  auto dma_u = [&](const void *to, const void *from) {
    const unsigned l = __builtin_amdgcn_readfirstlane((unsigned)(uintptr_t)(__attribute__((address_space(3))) void *)to);
    if constexpr (ONCE) asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2 nt" ::"s"(l), "v"(lane_off), "s"(from) : "memory");
    else asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2" ::"s"(l), "v"(lane_off), "s"(from) : "memory");
  };
  // slab fb: chunk (rb, s, hi / lo) = fragment (rb, fb, s) of either array; past the last one it is fetched again, so that
  // a request is always six loads
  auto request = [&](int fb, int slot) {
    const int src = min(fb, FB - 1);
#pragma unroll
    for (int x4 = 0; x4 < 4; ++x4) dma_u(&tile[((slot * 8 + w) * 4 + x4) * 64], usrc + (src * 4 + x4) * 64);
#pragma unroll
    for (int i = 0; i < RB * 4 / 8; ++i) {
      const int c = i * 8 + w;
      const bf16x8 *gp = ((c & 1) ? st_lo : st_hi) + (int64_t)bh * (D * F / 8) + (((c >> 2) * FB + src) * 2 + ((c >> 1) & 1)) * 64;
      dma(&ring[slot * SLOT + c * 64], gp);
    }
  };
  const WideOutStage os = wide_out_stage(stat, (int64_t)bh * n_tb + tb, F, act, P, lane);
  request(0, 0);
  request(1, 1);
  f32x16 acc[RB];
#pragma unroll
  for (int rb = 0; rb < RB; ++rb)
#pragma unroll
    for (int v = 0; v < 16; ++v) acc[rb][v] = 0.f;
  float dot = 0.f;
  int slot = 0;
#pragma unroll 1
  for (int fb = 0; fb < FB; ++fb) {
    asm volatile("s_waitcnt vmcnt(6)" ::: "memory");    // the request behind this tile's
    __syncthreads();                                    // this tile's slab is there, the last tile's slot is free
    request(fb + 2, slot == 0 ? 2 : slot - 1);
    const lds_frag_ptr sl = (lds_frag_ptr)&ring[slot * SLOT];
    f32x4 raw[4];
#pragma unroll
    for (int x4 = 0; x4 < 4; ++x4) raw[x4] = tile[((slot * 8 + w) * 4 + x4) * 64 + lane];
    bf16x8 b[2];
    wide_phi_tile(raw, fb, os, valid, b);
#pragma unroll
    for (int s = 0; s < 2; ++s) {
#pragma unroll
      for (int x = 0; x < 2; ++x) {
        const f32x4 z4 = *reinterpret_cast<const f32x4 *>(&zl[32 * fb + 16 * s + 8 * x + 4 * g]);
#pragma unroll
        for (int j = 0; j < 4; ++j) dot += static_cast<float>(b[s][4 * x + j]) * z4[j];
      }
#pragma unroll
      for (int lo = 1; lo >= 0; --lo)
#pragma unroll
        for (int rb = 0; rb < RB; ++rb) acc[rb] = mfma32(frag_at(sl, rb * 4 + s * 2 + lo, lane), b[s], acc[rb]);
    }
    slot = slot == 2 ? 0 : slot + 1;
  }
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");      // nothing may still be on its way into this workgroup's LDS
  if (!live) return;
  dot = xhalf_sum(dot);
  if (g == 0 && valid) e_out[(int64_t)bh * n_tok + 32 * tb + r] = dot;
#pragma unroll
  for (int rb = 0; rb < RB; ++rb)
#pragma unroll
    for (int x4 = 0; x4 < 4; ++x4)
      lin[((((int64_t)bh * n_tb + tb) * RB + rb) * 4 + x4) * 64 + lane] =
          f32x4{acc[rb][4 * x4], acc[rb][4 * x4 + 1], acc[rb][4 * x4 + 2], acc[rb][4 * x4 + 3]};
}

// ------------------------------------------------------------------------------------------------
// host side

template <typename T>
static inline T *ws_ptr(void *ws, size_t off) { return reinterpret_cast<T *>(static_cast<char *>(ws) + off); }
static inline size_t align256(size_t x) { return (x + 255) & ~static_cast<size_t>(255); }

void make_wide_plan(const Plan &pl, size_t base_off, WidePlan &wp, bool backward) {
  const size_t BH = (size_t)pl.B * pl.H;
  wp.n_tb_q = (pl.N + 31) / 32;
  wp.n_tb_k = (pl.NL + 31) / 32;
  const size_t n_tb = wp.n_tb_q;                      // the key side (fewer tokens) reuses the query side's buffers
  size_t off = base_off;
  auto take = [&](size_t bytes) { size_t o = off; off += align256(bytes); return o; };
  const int KL = pl.DM > 0 ? pl.DM : pl.HD;            // input width of the last layer
  wp.off_w1 = take((size_t)pl.H * pl.HD * pl.D * 2);
  wp.off_wm = take((size_t)pl.H * pl.DM * pl.HD * 2);
  wp.off_w2 = take((size_t)pl.H * pl.F * KL * 2);
  wp.off_hhi = take(backward ? BH * n_tb * 32 * pl.HD * 2 : 0);
  wp.off_h2hi = take(BH * n_tb * 32 * pl.DM * 2);
  wp.off_h2lo = take(BH * n_tb * 32 * pl.DM * 2);
  wp.off_u = take(BH * n_tb * 32 * (size_t)pl.F * 4);
  wp.off_stat = take(BH * n_tb * (pl.F / 128) * 2 * 64 * sizeof(float));
  wp.off_phi = take(backward ? BH * n_tb * 32 * (size_t)pl.F * 2 : 0);
  wp.off_lin = take(BH * n_tb * 32 * (size_t)pl.D * 4);
  wp.off_e = take(BH * (size_t)pl.N * 4);
  wp.total = off;
}

// One feature map over one token set: weight fragments, layer 1, (middle layer,) last layer, which leaves the fp32
// pre-activations and the softmax statistics; the output stage belongs to whoever reads them next.  is_query: all N
// tokens of q; otherwise the linear tokens of k.
hipError_t launch_wide_map(const Plan &pl, const WidePlan &wp, const void *x, const ha_feature_map &fm, bool is_query,
                           void *ws, hipStream_t st, bool keep_hidden) {
  const int n_tok = is_query ? pl.N : pl.NL;
  hipError_t e;
  const int KL = pl.DM > 0 ? pl.DM : pl.HD;
  // weight fragments of this map
  {
    WidePrepMap m;
    int n = 0, cols = 0;
    auto layer = [&](const void *w, size_t off, int nout, int kdim, bool chained) {
      m.layer[n++] = WidePrepLayer{w, ws_ptr<bf16x8>(ws, off), nout, kdim, cols, chained};
      cols += (nout * kdim / 8 + 255) / 256;
    };
    layer(fm.w1, wp.off_w1, pl.HD, pl.D, false);
    if (pl.DM > 0) layer(fm.w_mid, wp.off_wm, pl.DM, pl.HD, true);
    layer(fm.w2, wp.off_w2, pl.F, KL, true);
    if (n == 2) m.layer[2] = m.layer[1];
    const dim3 grid(cols, pl.H);
    if (pl.f32) wide_prep_kernel<true><<<grid, 256, 0, st>>>(m);
    else wide_prep_kernel<false><<<grid, 256, 0, st>>>(m);
    if ((e = hipGetLastError()) != hipSuccess) return e;
  }
  // x -> first hidden layer (-> middle layer, hi + lo images) -> fp32 pre-activations and softmax statistics
  WideMlpLayer l = {};
  l.x = x;
  l.n_tok = n_tok; l.R = is_query ? 0 : pl.R;
  l.w1f = ws_ptr<void>(ws, wp.off_w1);
  l.b1 = fm.b1;
  l.K = pl.HD;
  if (keep_hidden) l.h_hi = ws_ptr<void>(ws, wp.off_hhi);
  if (pl.DM > 0) {
    l.wf = ws_ptr<void>(ws, wp.off_wm);
    l.bias = fm.b_mid;
    l.NOUT = pl.DM;
    l.out_hi = ws_ptr<void>(ws, wp.off_h2hi);
    l.out_lo = ws_ptr<void>(ws, wp.off_h2lo);
    if ((e = launch_wide_mlp(pl, l, st)) != hipSuccess) return e;
    l.x = nullptr;
    l.h_hi = nullptr;
    l.in_hi = l.out_hi; l.in_lo = l.out_lo;
    l.out_hi = l.out_lo = nullptr;
    l.K = pl.DM;
  }
  l.wf = ws_ptr<void>(ws, wp.off_w2);
  l.bias = fm.b2;
  l.NOUT = pl.F;
  l.out_u = ws_ptr<void>(ws, wp.off_u);
  l.out_stat = ws_ptr<float>(ws, wp.off_stat);
  l.channel_lanes = !is_query && !keep_hidden;         // (a backward pass reads a token per lane, as the query side does)
  return launch_wide_mlp(pl, l, st);
}

// Pre-activations that the memory-side cache cannot hold between the writer and its reader are read non-temporally, so that they do
// not displace what is still to be read; from a quarter above its size on, because below that the parts still in it are worth more.
// Forward, cached / non-temporal: 12 heads, 8 blocks, 768 wide, 1.2 GB 4678 / 4660 us; 512 wide, 491 MB 974 / 946; 384 wide, 368 MB
// 1250 / 1222; 768 wide, 307 MB 899 / 904; 512 wide, 38 MB 153 / 156.
static bool wide_read_once(const Plan &pl, int n_tb) {
  return (int64_t)pl.B * pl.H * n_tb * 32 * pl.F * 4 > kMemorySideCache + kMemorySideCache / 4;
}

// Key side: phi_k over the linear tokens, then [S | z] (partials + the forward's reduction).
hipError_t launch_wide_key_side(const Plan &pl, const WidePlan &wp, const void *k, const void *v, const ha_feature_map &phi_k,
                                void *ws, hipStream_t st) {
  hipError_t e = launch_wide_map(pl, wp, k, phi_k, false, ws, st, false);
  if (e != hipSuccess) return e;
  // eight row blocks per workgroup where the width has them: V is fetched for half as many, and a barrier serves twice the work
  const int n_pairs = pl.n_chunks * pl.B * pl.H, nw = pl.F % 256 == 0 ? 8 : 4;
  const dim3 grid((n_pairs + 7) / 8 * 8 * (pl.F / 32 / nw));
  const bool once = wide_read_once(pl, wp.n_tb_k);
#define HA_WIDE_STATE(NW, F32) \
  (once ? wide_state_kernel<NW, F32, true> : wide_state_kernel<NW, F32, false>)<<<grid, 64 * NW, 0, st>>>(ws_ptr<f32x4>(ws, wp.off_u), ws_ptr<float>(ws, wp.off_stat), v, \
                                                       ws_ptr<float>(ws, pl.off_part), pl.H, pl.NL, pl.R, pl.G, pl.CH, pl.F, \
                                                       wp.n_tb_k, pl.act_k, pl.P, pl.sb, pl.sh, pl.sn, pl.n_chunks, n_pairs)
  if (nw == 8) { if (pl.f32) HA_WIDE_STATE(8, true); else HA_WIDE_STATE(8, false); }
  else { if (pl.f32) HA_WIDE_STATE(4, true); else HA_WIDE_STATE(4, false); }
#undef HA_WIDE_STATE
  if ((e = hipGetLastError()) != hipSuccess) return e;
  return launch_state_reduce(pl, ws, st);
}

// Query side: phi_q over all tokens, e = phi_q . z, n = phi_q S; the query kernel picks both up in its epilogue.
hipError_t launch_wide_query_side(const Plan &pl, const WidePlan &wp, const void *q, const ha_feature_map &phi_q, void *ws,
                                  hipStream_t st) {
  hipError_t e = launch_wide_map(pl, wp, q, phi_q, true, ws, st, false);
  if (e != hipSuccess) return e;
  dim3 grid((wp.n_tb_q + 7) / 8, pl.B * pl.H);
  (wide_read_once(pl, wp.n_tb_q) ? wide_lin_kernel<128, true> : wide_lin_kernel<128, false>)<<<grid, 512, 0, st>>>(ws_ptr<f32x4>(ws, wp.off_u), ws_ptr<float>(ws, wp.off_stat),
                                             ws_ptr<bf16x8>(ws, pl.off_sthi), ws_ptr<bf16x8>(ws, pl.off_stlo),
                                             ws_ptr<float>(ws, pl.off_z), ws_ptr<f32x4>(ws, wp.off_lin),
                                             ws_ptr<float>(ws, wp.off_e), pl.F, pl.N, wp.n_tb_q, pl.act_q, pl.P);
  return hipGetLastError();
}

}  // namespace ha
