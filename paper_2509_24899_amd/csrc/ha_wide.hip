// Feature maps of any width (Attention Surgery, Sec. 3.2 "Characterization of phi"; Tab. "phi": d -> P d -> P d
// for P = 2, 3, 4 and the three-layer P = 6 map), gfx950.  The fused kernels keep a token's hidden activations and
// all its output channels in registers, which ends at 256 channels.  Here every layer is a pass of its own and
// activations travel through HBM, in exactly the register image the next product wants:
//
//   wide_prep_kernel       one weight matrix -> A-operand fragments (natural order for layer 1, chained after it)
//   (ha_wide_mlp.hip)      h^T = relu(W1 x^T + b1) on the way into  h'^T = relu(W h^T + b)  or  u^T = W h^T + b  (last
//                          layer: fp32 pre-activations); h' as hi + lo bf16
//   (output stage)         softmax / exp / relu over all channels of a token, slice powers, bf16: applied by the two
//                          consumers below while they read the pre-activations, so phi never visits HBM
//   wide_state_kernel      [S | z] += phi_k^T [V | 1], one 128-channel slab of S per workgroup
//   wide_lin_kernel        n_i = phi_q(q_i) S   (fp32, in the layout of the query kernel's accumulators), e_i = phi_q(q_i).z
// The query kernel then adds n_i and e_i in its epilogue instead of evaluating phi_q itself.
//
// Register images ("C image" of a 32-token block tb of (batch, head) bh; lane = 32 g + r owns token 32 tb + r):
//   activations   bf16x8 [bh][tb][W/32][2][64]   piece (block c, half s) = channels 32 c + crow(8 s + t, g), t = 0..7,
//                                                i.e. the B operand ("chained" order) of the next product
//   fp32 tiles    f32x4  [bh][tb][W/32][4][64]   piece (block c, quad x) = channels 32 c + crow(4 x + j, g), j = 0..3
#include "ha_device.h"
#include "ha_plan.h"

namespace ha {

// ------------------------------------------------------------------------------------------------
// wide_prep_kernel: grid (ceil(NOUT*K / 2048), H).  W [H][NOUT][K] (io dtype) -> fragments, see weight_piece
template <bool F32, bool CHAINED>
__global__ __launch_bounds__(256) void wide_prep_kernel(const void *__restrict__ wsrc, bf16x8 *__restrict__ wf, int NOUT, int K) {
  const int piece = blockIdx.x * 256 + threadIdx.x;
  const int64_t n = (int64_t)NOUT * K, base = blockIdx.y * n;
  if (piece < n / 8) wf[base / 8 + piece] = weight_piece<F32, CHAINED>(wsrc, base, K, piece);
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
static __device__ __forceinline__ void wide_load_tile(const f32x4 *__restrict__ src, int fb, f32x4 (&raw)[4]) {
#pragma unroll
  for (int x4 = 0; x4 < 4; ++x4) raw[x4] = src[(fb * 4 + x4) * 64];
}
static __device__ __forceinline__ void wide_phi_tile(const f32x4 *__restrict__ src, int fb, const WideOutStage &o, bool valid,
                                                     bf16x8 (&out)[2]) {
  f32x4 raw[4];
  wide_load_tile(src, fb, raw);
  wide_phi_tile(raw, fb, o, valid, out);
}

// ------------------------------------------------------------------------------------------------
// wide_state_kernel: grid (n_chunks, B*H, F / 128), 4 waves.  As the contraction half of state_kernel, with
// phi_k formed from the fp32 pre-activations of the last layer as they are read; workgroup z owns feature rows
// 128 z .. 128 z + 127 of [S | z], wave w row block w of those.  Partial tiles go where state_kernel puts them
// (part[bh][chunk][row block * NCB + column block][v][lane]), so state_reduce_kernel serves both.
template <int D, bool F32>
__global__ __launch_bounds__(256, 1) void wide_state_kernel(const f32x4 *__restrict__ u_img, const float *__restrict__ stat,
                                                            const void *__restrict__ v, float *__restrict__ part, int H,
                                                            int NL, int R, int G, int CH, int F, int n_tb, int act, int P,
                                                            int64_t sb, int64_t sh, int64_t sn) {
  constexpr int TOK = 128, PITCH = TOK + 8, NCB = D / 32 + 1;
  constexpr int CG = D / 32, VPT = (TOK / 16) * CG / 4;
  __shared__ __align__(16) __bf16 ft[128][PITCH];
  __shared__ __align__(16) __bf16 vt[D][PITCH];
  const int chunk = blockIdx.x, bh = blockIdx.y, zb = blockIdx.z, h = bh % H;
  const int64_t base = (int64_t)(bh / H) * sb + (int64_t)h * sh;
  const int tid = threadIdx.x, lane = tid & 63, r = lane & 31, g = lane >> 5;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int FB = F / 32;
  const LinearMap lmap(R, G);
  f32x16 acc[NCB];
#pragma unroll
  for (int i = 0; i < NCB; ++i)
#pragma unroll
    for (int x = 0; x < 16; ++x) acc[i][x] = 0.f;
  const int tf = w * 32 + r;
  int fcol[4];
#pragma unroll
  for (int q = 0; q < 4; ++q) fcol[q] = (4 * g) * PITCH + ((((tf >> 3) ^ (2 * q)) << 3) | (tf & 7));
  const int vsw = (lane >> 4) << 1;
  const int vrow0 = 8 * (lane >> 4) * PITCH;
  const int rsw = ((r >> 3) & 3) << 1;
  __bf16 *ftp = &ft[0][0];
  __bf16 *vtp = &vt[0][0];
  const __bf16 one = static_cast<__bf16>(r == 0 ? 1.0f : 0.0f);
  const bf16x8 ones = bf16x8{one, one, one, one, one, one, one, one};
  const int lt_begin = chunk * CH, lt_end = min(lt_begin + CH, NL);
  for (int t0 = lt_begin; t0 < lt_end; t0 += TOK) {
    bf16x8 vreg[VPT];
#pragma unroll
    for (int p = 0; p < VPT; ++p) {
      const int trow = 16 * ((4 * p + w) & 7) + (lane & 15), c8 = 4 * (p >> 1) + (lane >> 4);
      const int tok = lmap.token(min(t0 + trow, NL - 1));
      vreg[p] = load8<F32>(v, base + (int64_t)tok * sn + c8 * 8);
    }
    const int tb = min(t0 / 32 + w, n_tb - 1);            // blocks past the end: clamped, their tokens are not valid
    const bool valid = t0 + tf < NL;
    const WideOutStage os = wide_out_stage(stat, (int64_t)bh * n_tb + tb, F, act, P, lane);
    const f32x4 *usrc = u_img + ((int64_t)bh * n_tb + tb) * FB * 256 + lane;
    bf16x8 ph[4][2];
#pragma unroll
    for (int fb = 0; fb < 4; ++fb) wide_phi_tile(usrc, 4 * zb + fb, os, valid, ph[fb]);
#pragma unroll
    for (int fb = 0; fb < 4; ++fb)
#pragma unroll
      for (int x = 0; x < 16; ++x) ftp[(32 * fb + 8 * (x >> 2) + (x & 3)) * PITCH + fcol[x >> 2]] = ph[fb][x >> 3][x & 7];
#pragma unroll
    for (int p = 0; p < VPT; ++p) {
      const int trow = 16 * ((4 * p + w) & 7) + (lane & 15);
      const int col = (((trow >> 3) ^ vsw) << 3) | (trow & 7);
#pragma unroll
      for (int i = 0; i < 8; ++i) vtp[(32 * (p >> 1) + i) * PITCH + vrow0 + col] = vreg[p][i];
    }
    __syncthreads();
#pragma unroll
    for (int ks = 0; ks < TOK / 16; ++ks) {
      const int col = ((2 * ks + g) ^ rsw) << 3;
      const bf16x8 af = *reinterpret_cast<const bf16x8 *>(&ftp[(32 * w + r) * PITCH + col]);
#pragma unroll
      for (int cb = 0; cb < NCB; ++cb) {
        const bf16x8 bfr = cb < D / 32 ? *reinterpret_cast<const bf16x8 *>(&vtp[(32 * cb + r) * PITCH + col]) : ones;
        acc[cb] = mfma32(af, bfr, acc[cb]);
      }
    }
    __syncthreads();
  }
  float *dst = part + (((int64_t)bh * gridDim.x + chunk) * FB + 4 * zb + w) * NCB * 1024;
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
// (every wave reading its own from L2, 4.7 GB of them: 460 us at 480p / 81 frames, 768 wide, 12 heads; now 355).  The
// wave's own tile of pre-activations comes with it, two tiles ahead: the bound is HBM, 1.2 GB of them, and 64 KiB per CU
// are on their way.
// All loads of the loop are LDS-DMA so that the counts below are the only waits.
template <int D>
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
  // slab fb: chunk (rb, s, hi / lo) = fragment (rb, fb, s) of either array; past the last one it is fetched again, so that
  // a request is always six loads
  auto request = [&](int fb, int slot) {
    const int src = min(fb, FB - 1);
#pragma unroll
    for (int x4 = 0; x4 < 4; ++x4) dma(&tile[((slot * 8 + w) * 4 + x4) * 64], usrc + (src * 4 + x4) * 64);
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
    auto prep = [&](const void *wsrc, size_t off, int nout, int kdim, bool chained) {
      dim3 grid((nout * kdim / 8 + 255) / 256, pl.H);
      bf16x8 *dst = ws_ptr<bf16x8>(ws, off);
      if (pl.f32) {
        if (chained) wide_prep_kernel<true, true><<<grid, 256, 0, st>>>(wsrc, dst, nout, kdim);
        else wide_prep_kernel<true, false><<<grid, 256, 0, st>>>(wsrc, dst, nout, kdim);
      } else {
        if (chained) wide_prep_kernel<false, true><<<grid, 256, 0, st>>>(wsrc, dst, nout, kdim);
        else wide_prep_kernel<false, false><<<grid, 256, 0, st>>>(wsrc, dst, nout, kdim);
      }
    };
    prep(fm.w1, wp.off_w1, pl.HD, pl.D, false);
    if (pl.DM > 0) prep(fm.w_mid, wp.off_wm, pl.DM, pl.HD, true);
    prep(fm.w2, wp.off_w2, pl.F, KL, true);
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
  return launch_wide_mlp(pl, l, st);
}

// Key side: phi_k over the linear tokens, then [S | z] (partials + the forward's reduction).
hipError_t launch_wide_key_side(const Plan &pl, const WidePlan &wp, const void *k, const void *v, const ha_feature_map &phi_k,
                                void *ws, hipStream_t st) {
  hipError_t e = launch_wide_map(pl, wp, k, phi_k, false, ws, st, false);
  if (e != hipSuccess) return e;
  dim3 grid(pl.n_chunks, pl.B * pl.H, pl.F / 128);
  if (pl.f32)
    wide_state_kernel<128, true><<<grid, 256, 0, st>>>(ws_ptr<f32x4>(ws, wp.off_u), ws_ptr<float>(ws, wp.off_stat), v,
                                                       ws_ptr<float>(ws, pl.off_part), pl.H, pl.NL, pl.R, pl.G, pl.CH, pl.F,
                                                       wp.n_tb_k, pl.act_k, pl.P, pl.sb, pl.sh, pl.sn);
  else
    wide_state_kernel<128, false><<<grid, 256, 0, st>>>(ws_ptr<f32x4>(ws, wp.off_u), ws_ptr<float>(ws, wp.off_stat), v,
                                                        ws_ptr<float>(ws, pl.off_part), pl.H, pl.NL, pl.R, pl.G, pl.CH, pl.F,
                                                        wp.n_tb_k, pl.act_k, pl.P, pl.sb, pl.sh, pl.sn);
  if ((e = hipGetLastError()) != hipSuccess) return e;
  return launch_state_reduce(pl, ws, st);
}

// Query side: phi_q over all tokens, e = phi_q . z, n = phi_q S; the query kernel picks both up in its epilogue.
hipError_t launch_wide_query_side(const Plan &pl, const WidePlan &wp, const void *q, const ha_feature_map &phi_q, void *ws,
                                  hipStream_t st) {
  hipError_t e = launch_wide_map(pl, wp, q, phi_q, true, ws, st, false);
  if (e != hipSuccess) return e;
  dim3 grid((wp.n_tb_q + 7) / 8, pl.B * pl.H);
  wide_lin_kernel<128><<<grid, 512, 0, st>>>(ws_ptr<f32x4>(ws, wp.off_u), ws_ptr<float>(ws, wp.off_stat),
                                             ws_ptr<bf16x8>(ws, pl.off_sthi), ws_ptr<bf16x8>(ws, pl.off_stlo),
                                             ws_ptr<float>(ws, pl.off_z), ws_ptr<f32x4>(ws, wp.off_lin),
                                             ws_ptr<float>(ws, wp.off_e), pl.F, pl.N, wp.n_tb_q, pl.act_q, pl.P);
  return hipGetLastError();
}

}  // namespace ha
