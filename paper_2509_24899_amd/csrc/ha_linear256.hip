// Query side of the linear part for the maps 128 -> 256 -> 256 (the paper's default widths, Tab. "phi", P = 2):
//     n_i = phi_q(q_i) S   and   e_i = phi_q(q_i) . z
// for all queries, n as the fp32 register image the query kernel adds to its accumulators (see wide_lin_kernel), e per
// query.  gfx950 only.
//
// As the query kernel's epilogue this costs 57 us per round of workgroups at 480p / 81 frames (340 us of 1627): hidden
// activations, accumulators and features of 256 channels do not fit the registers the softmax accumulators leave, and the
// operands (W1 64 KiB, W2 128 KiB, S hi + lo 128 KiB per head) pass through the ring in three exposed rounds.  Here the map is
// evaluated a hidden block at a time (ha_mlp256.h), and the operands stream through an LDS ring in that very order, 24 KiB per hidden block, then 16 KiB
// per feature block of S; the stream runs ahead over the tiles and heads of a workgroup, one barrier per slab.
//
// Bound: matrix cores, 448 instructions of 32 cycles per 32-query block (28.7 k cycles per 256-query tile), next to 9 k
// cycles of exponentials and packing and the conversion of each hidden block, which the barrier keeps both waves of a SIMD
// in at the same time (matrix cores busy for 45 % of the cycles at 2.06 GHz); n costs 201 MB written here and read again.  Measured at 480p / 81 frames, 12 heads: this pass 174 us (178 with the features rounded tile by tile)
// and the query kernel 1413 us where the query kernel alone took 1627 on a faster box (forward 1959 -> 1858 us side by
// side); B = 2, H = 12, N = 5003, fp32, R = 3: 198 us -> 79 + 127 us in a round and a half less exposed epilogue (355 -> 329
// us); the fixed cost of a small call falls from 64 to about 25 us.
#include "ha_device.h"
#include "ha_mlp256.h"
#include "ha_plan.h"

namespace ha {

struct Linear256Args {
  const void *q;
  const bf16x8 *w1f, *w2f;               // phi_q fragments, per head
  const float *b1, *b2;                  // phi_q biases, per head (may be null)
  const bf16x8 *st_hi, *st_lo;           // [B*H][D/32][F/32][2][64]
  const float *z;                        // [B*H][F]
  f32x4 *lin;                            // [B*H][n_tb][D/32][4][64]
  float *e_out;                          // [B*H][N]
  int H, N, P, act, n_tb;                // n_tb: 32-query blocks per (batch, head), a whole number of tiles
  int n_tiles, total;                    // tiles of 32 NW queries per (batch, head), and overall
  int64_t sb, sh, sn;
};

// NW waves of 32 queries per tile, NBUF slabs in the ring.  Grid: persistent, workgroups take contiguous runs of tiles, and
// the workgroups of one XCD (blockIdx % 8) neighbouring runs, so an XCD's L2 holds the operands of few heads.
template <int NW, int NBUF, bool F32, bool ACT0, bool P2>
__global__ __launch_bounds__(64 * NW, 2) void linear256_kernel(Linear256Args a) {
  constexpr int D = 128, HD = 256, F = 256, KS = D / 16, HB = HD / 32, FB = F / 32, RB = D / 32;
  constexpr int WCH = kSlabChunks, SCH = RB * 4;          // 1 KiB chunks per slab: of the weights, of S
  constexpr int SLOT = WCH * 64, STEPS = HB + FB;
  constexpr int NW1 = HD * D / 8, NW2 = F * HD / 8, NST = D * F / 8;
  static_assert(NBUF >= 3 && NBUF <= STEPS && WCH % NW == 0 && SCH % NW == 0, "slabs are dealt evenly");
  __shared__ bf16x8 ring[NBUF * SLOT];
  __shared__ __align__(16) float vecs[HD + 2 * F];        // b1, b2, z
  const int tid = threadIdx.x, lane = tid & 63, r = lane & 31, g = lane >> 5;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int nwg = gridDim.x;                              // a multiple of 8
  const int wg = (blockIdx.x & 7) * (nwg >> 3) + (blockIdx.x >> 3);
  const int t_lo = (int)((int64_t)wg * a.total / nwg), t_hi = (int)((int64_t)(wg + 1) * a.total / nwg);
  if (t_lo >= t_hi) return;

  // slab `s` of a tile of (batch, head) bh -> ring slot; chunks are dealt round-robin to the waves
  const unsigned lane_off = lane * 16;
  auto request = [&](int bh, int s, int slot) {
    const int h = bh % a.H;
    const bool weights = s < HB;
    auto dma = [&](const bf16x8 *gp, int c) {
      const unsigned l = __builtin_amdgcn_readfirstlane(
          (unsigned)(uintptr_t)(__attribute__((address_space(3))) void *)(&ring[slot * SLOT + c * 64]));
      asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2" ::"s"(l), "v"(lane_off), "s"(gp) : "memory");
    };
    if (weights) {
#pragma unroll
      for (int i = 0; i < WCH / NW; ++i) {
        const int c = i * NW + w;
        dma(slab_chunk(a.w1f + (int64_t)h * NW1, a.w2f + (int64_t)h * NW2, s, c), c);
      }
    } else {
#pragma unroll
      for (int i = 0; i < SCH / NW; ++i) {
        const int c = i * NW + w;                         // (row block, half, hi / lo) of feature block s - HB
        const bf16x8 *gp = ((c & 1) ? a.st_lo : a.st_hi) + (int64_t)bh * NST + (((c >> 2) * FB + s - HB) * 2 + ((c >> 1) & 1)) * 64;
        dma(gp, c);
      }
    }
  };
  // Barrier ahead of a slab: this wave's share of it has landed and so has everybody's, and everybody is done with the slab
  // before it, whose slot takes the request NBUF - 1 slabs ahead.  At least SCH / NW requests per newer slab may stay in
  // flight (loads and stores retire in order), and in the first NBUF - 1 slabs after a tile's output also its 4 RB stores.
  constexpr int FLY = (NBUF - 2) * (SCH / NW);
  static_assert(FLY + 4 * RB < 63, "vmcnt immediate too large");
  int slot = 0, ahead = NBUF - 1;                         // slot of the current slab; slot the next request goes to
  int bh = t_lo / a.n_tiles, bh_next = bh;
  auto advance = [&](int step, bool after_output) {
    if (after_output && step < NBUF - 1) asm volatile("s_waitcnt vmcnt(%0)" ::"n"(FLY + 4 * RB) : "memory");
    else asm volatile("s_waitcnt vmcnt(%0)" ::"n"(FLY) : "memory");
    __syncthreads();
    const int s = step + NBUF - 1;
    request(s < STEPS ? bh : bh_next, s < STEPS ? s : s - STEPS, ahead);   // (past the last tile: slabs nobody reads)
    ahead = ahead + 1 == NBUF ? 0 : ahead + 1;
  };
  auto load_q = [&](int t, bf16x8 (&dst)[KS]) {
    const int b = t / a.n_tiles, hh = b % a.H;
    const int64_t base = (int64_t)(b / a.H) * a.sb + (int64_t)hh * a.sh;
    const int qi = min((t - b * a.n_tiles) * 32 * NW + 32 * w + r, a.N - 1);   // rows past the end repeat the last query
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) dst[ks] = load8<F32>(a.q, base + (int64_t)qi * a.sn + 16 * ks + 8 * g);
  };
  bf16x8 xf[KS];
  load_q(t_lo, xf);
#pragma unroll
  for (int s = 0; s < NBUF - 1; ++s) request(bh, s, s);
  const float *b1 = &vecs[0], *b2 = &vecs[HD], *zz = &vecs[HD + F];

  int bh_vecs = -1;
  for (int t = t_lo; t < t_hi; ++t) {
    bh_next = t + 1 < t_hi ? (t + 1) / a.n_tiles : bh;
    if (bh != bh_vecs) {                                  // workgroup-uniform: the first tile, or the head changes
      const int h = bh % a.H;
      __syncthreads();                                    // every wave is done with the previous head's vectors
      for (int i = tid; i < HD; i += 64 * NW) vecs[i] = a.b1 ? a.b1[(int64_t)h * HD + i] : 0.f;
      for (int i = tid; i < F; i += 64 * NW) vecs[HD + i] = a.b2 ? a.b2[(int64_t)h * F + i] : 0.f;
      for (int i = tid; i < F; i += 64 * NW) vecs[HD + F + i] = a.z[(int64_t)bh * F + i];
      bh_vecs = bh;
      __syncthreads();
    }
    // ---------------- the map: u = W2 relu(W1 x + b1) + b2, one hidden block per slab
    f32x16 u[FB];
#pragma unroll
    for (int fb = 0; fb < FB; ++fb) u[fb] = column_tile(b2, fb, g);
#pragma unroll 1
    for (int hb = 0; hb < HB; ++hb) {
      advance(hb, t > t_lo);
      const lds_frag_ptr sl = (lds_frag_ptr)&ring[slot * SLOT];
      slot = slot + 1 == NBUF ? 0 : slot + 1;
      mlp256_hidden_block(sl, b1, hb, xf, lane, g, u);
    }
    load_q(t + 1 < t_hi ? t + 1 : t, xf);                 // the next tile's rows travel under everything below
    // ---------------- output stage: positive activation over all channels, slice powers, bf16
    phi256_output<ACT0, P2>(u, a.act, a.P);
    u32x4 gb[FB][2];                                      // word i of half s: channels crow(8 s + 2 i, g) and the next
#pragma unroll
    for (int fb = 0; fb < FB; ++fb) {
#pragma unroll
      for (int s = 0; s < 2; ++s)
#pragma unroll
        for (int i = 0; i < 4; ++i) gb[fb][s][i] = pack_bf16(u[fb][8 * s + 2 * i], u[fb][8 * s + 2 * i + 1]);
    }
    // ---------------- n^T = S^T phi^T and e = phi . z (from the rounded phi), one feature block per slab
    f32x16 n[RB];
#pragma unroll
    for (int rb = 0; rb < RB; ++rb)
#pragma unroll
      for (int x = 0; x < 16; ++x) n[rb][x] = 0.f;
    float e = 0.f;
#pragma unroll
    for (int fb = 0; fb < FB; ++fb) {
      advance(HB + fb, false);
      const lds_frag_ptr sl = (lds_frag_ptr)&ring[slot * SLOT];
      slot = slot + 1 == NBUF ? 0 : slot + 1;
#pragma unroll
      for (int s = 0; s < 2; ++s) {
        const bf16x8 b8 = __builtin_bit_cast(bf16x8, gb[fb][s]);
#pragma unroll
        for (int lo = 1; lo >= 0; --lo)
#pragma unroll
          for (int rb = 0; rb < RB; ++rb) n[rb] = mfma32(frag_at(sl, rb * 4 + s * 2 + lo, lane), b8, n[rb]);
#pragma unroll
        for (int q = 0; q < 2; ++q) {
          const f32x4 z4 = *reinterpret_cast<const f32x4 *>(zz + 32 * fb + 16 * s + 8 * q + 4 * g);
#pragma unroll
          for (int j = 0; j < 4; j += 2) {
            const unsigned pair = gb[fb][s][2 * q + j / 2];
            e = __builtin_fmaf(__uint_as_float(pair << 16), z4[j], e);
            e = __builtin_fmaf(__uint_as_float(pair & 0xffff0000u), z4[j + 1], e);
          }
        }
      }
    }
    e = xhalf_sum(e);
    const int tb = (t - bh * a.n_tiles) * NW + w, qi = 32 * tb + r;
    if (g == 0 && qi < a.N) a.e_out[(int64_t)bh * a.N + qi] = e;
#pragma unroll
    for (int rb = 0; rb < RB; ++rb)
#pragma unroll
      for (int x4 = 0; x4 < 4; ++x4)
        a.lin[((((int64_t)bh * a.n_tb + tb) * RB + rb) * 4 + x4) * 64 + lane] =
            f32x4{n[rb][4 * x4], n[rb][4 * x4 + 1], n[rb][4 * x4 + 2], n[rb][4 * x4 + 3]};
    bh = bh_next;
  }
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");        // nothing may still be on its way into this workgroup's LDS
}

hipError_t launch_linear256(const Plan &pl, const void *q, const ha_feature_map &phi_q, void *ws, hipStream_t st) {
  char *wsb = static_cast<char *>(ws);
  Linear256Args a;
  a.q = q;
  a.w1f = reinterpret_cast<bf16x8 *>(wsb + pl.off_w1q);
  a.w2f = reinterpret_cast<bf16x8 *>(wsb + pl.off_w2q);
  a.b1 = phi_q.b1;
  a.b2 = phi_q.b2;
  a.st_hi = reinterpret_cast<bf16x8 *>(wsb + pl.off_sthi);
  a.st_lo = reinterpret_cast<bf16x8 *>(wsb + pl.off_stlo);
  a.z = reinterpret_cast<float *>(wsb + pl.off_z);
  a.lin = reinterpret_cast<f32x4 *>(wsb + pl.off_lin);
  a.e_out = reinterpret_cast<float *>(wsb + pl.off_e);
  a.H = pl.H; a.N = pl.N; a.P = pl.P; a.act = pl.act_q; a.n_tb = pl.n_tb;
  a.sb = pl.sb; a.sh = pl.sh; a.sn = pl.sn;
  const int64_t BH = (int64_t)pl.B * pl.H;
  // Large tiles share one fetch of the operands (320 KiB) among 256 queries, one workgroup per CU; small ones, two
  // workgroups per CU, give a problem that has fewer than 256 large ones twice the workgroups.
  const bool big = (pl.N + 255) / 256 * BH >= 256;
  a.n_tiles = (pl.N + (big ? 255 : 127)) / (big ? 256 : 128);
  a.total = (int)(a.n_tiles * BH);
  const int most = big ? 256 : 512;                       // workgroups on the chip at once
  const int nwg = a.total < most ? (a.total + 7) / 8 * 8 : most;
#define HA_LIN256(F32, ACT0, P2) \
  do { \
    if (big) linear256_kernel<8, 6, F32, ACT0, P2><<<nwg, 512, 0, st>>>(a); \
    else linear256_kernel<4, 3, F32, ACT0, P2><<<nwg, 256, 0, st>>>(a); \
  } while (0)
#define HA_LIN256_MAP(F32) \
  do { \
    if (pl.act_q != HA_ACT_SOFTMAX) HA_LIN256(F32, false, false); \
    else if (pl.P == 2) HA_LIN256(F32, true, true); \
    else HA_LIN256(F32, true, false); \
  } while (0)
  if (pl.f32) HA_LIN256_MAP(true); else HA_LIN256_MAP(false);
#undef HA_LIN256_MAP
#undef HA_LIN256
  return hipGetLastError();
}

}  // namespace ha
