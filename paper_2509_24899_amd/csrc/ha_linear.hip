// Query side of purely linear attention (rate 0: no softmax tokens; Sec. 3.1) for the widths 128 -> 128 -> 128:
//     y_i = phi_q(q_i) S / (phi_q(q_i) . z),   gfx950 only,
// and, for small problems with softmax tokens, its numerator and denominator alone, which the query kernel adds.
//
// The query kernel of ha_query.hip runs this as its epilogue: every workgroup fetches the operands for one tile of 256
// queries, its waves go through load, layers, contraction and store in step, and memory is idle while they compute.
// With no softmax loop ahead of it that is the whole kernel, so here one workgroup per CU stays: W1, W2 and S (hi + lo)
// of one (batch, head) are 128 KiB, are fetched once and live in LDS, and each of the eight waves walks blocks of 32
// queries of its own with no barrier after the start.  The rows of the next block travel under layer 2 and everything
// behind it, the waves drift apart and one wave's stores and vector work sit under another's matrix instructions.
//
// Bound: the matrix cores.  160 matrix instructions of 32 cycles per 32-query block, two waves per SIMD: 10.2 k cycles per
// pair of blocks, of which the walk takes 12 k (cycle stamps) once the operands are there (9.5 k cycles after the start),
// at the 1.65 GHz the part sustains under this load; HBM (512 B per token and head) would take 40 us at the rate of a
// large copy.  Measured at 480p / 81 frames, 12 heads: 106 us in the query kernel, 78 us here with the contraction left to
// the compiler, 71 us with it in alternating pairs of row blocks, the denominator and the output of the first pair placed
// under the matrix instructions and a third of the vector instructions gone (whole forward 181 -> 148 us).  Operand
// fragments requested two steps ahead instead of one change nothing.
#include "ha_device.h"
#include "ha_mlp128.h"
#include "ha_plan.h"

namespace ha {

struct LinearArgs {
  const void *q;
  void *out;
  const bf16x8 *w1f, *w2f;               // phi_q fragments, per head
  const float *b1, *b2;                  // phi_q biases, per head (may be null)
  const bf16x8 *st_hi, *st_lo;           // [B*H][D/32][F/32][2][64]
  const float *z;                        // [B*H][F]
  float *row_den;                        // optional [B*H][N]
  int H, N, P, act;
  int64_t sb, sh, sn;
  f32x4 *lin;                            // PART: n^T as [B*H][n_tb][D/32][4][64], e as [B*H][N], instead of out
  float *lin_e;
  int n_tb;
  int per_bh, total;                     // workgroups per (batch, head), and overall
};

// grid: total, rounded up to a multiple of 8, 8 waves.  Consecutive workgroups of one XCD (blockIdx % 8) share a (batch, head),
// so that an XCD's L2 fetches the operands of an eighth of the heads and not of all (whole calls at rate 0 with one or two blocks
// per wave, us, before / after: H = 32, N = 1526  44.4 / 38.9; H = 24, N = 2038  41.0 / 37.4; H = 12, N = 3318  35.7 / 34.3;
// longer sequences the same).  ACT0: the output activation is the softmax over the channels; P2: the
// degree is 2, the paper's default (a branch on it here costs a copy of all feature registers).
template <bool F32, bool ACT0, bool P2, bool PART>
__global__ __launch_bounds__(512, 1) void linear_query_kernel(LinearArgs a) {
  constexpr int D = 128, F = 128, KS = D / 16, FB = F / 32, RB = D / 32, NOP = D * D / 8;
  // output staging, per wave: 32 query rows x 64 bytes (32 bf16 or 16 fp32 channels), rows padded by 16 bytes
  constexpr int PITCH = 64 + 16, ESZ = F32 ? 4 : 2, CPP = 64 / ESZ;
  __shared__ bf16x8 ops[4 * NOP];                        // W1, W2, S^T hi, S^T lo
  __shared__ __align__(16) float vecs[3 * F];            // b1, b2, z
  __shared__ __align__(16) char stage_all[8 * 32 * PITCH];
  const int per_xcd = (a.total + 7) >> 3, logical = (blockIdx.x & 7) * per_xcd + (blockIdx.x >> 3);
  if (logical >= a.total) return;
  const int bh = logical / a.per_bh, piece = logical % a.per_bh, h = bh % a.H;
  const int64_t base = (int64_t)(bh / a.H) * a.sb + (int64_t)h * a.sh;
  const int tid = threadIdx.x, lane = tid & 63, r = lane & 31, g = lane >> 5;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  dma_to_lds(a.w1f + (int64_t)h * NOP, &ops[0], NOP / 64, w, 8, lane);
  dma_to_lds(a.w2f + (int64_t)h * NOP, &ops[NOP], NOP / 64, w, 8, lane);
  dma_to_lds(a.st_hi + (int64_t)bh * NOP, &ops[2 * NOP], NOP / 64, w, 8, lane);
  dma_to_lds(a.st_lo + (int64_t)bh * NOP, &ops[3 * NOP], NOP / 64, w, 8, lane);
  if (tid < F) {
    vecs[tid] = a.b1 ? a.b1[(int64_t)h * F + tid] : 0.f;
    vecs[F + tid] = a.b2 ? a.b2[(int64_t)h * F + tid] : 0.f;
    vecs[2 * F + tid] = a.z[(int64_t)bh * F + tid];
  }
  // blocks of 32 queries of this workgroup, dealt to its waves
  const int nb = (a.N + 31) / 32;
  const int b_lo = (int)((int64_t)piece * nb / a.per_bh), b_hi = (int)((int64_t)(piece + 1) * nb / a.per_bh);
  auto load_q = [&](int blk, bf16x8 (&dst)[KS]) {
    const int qi = min(32 * blk + r, a.N - 1);           // rows past the end repeat the last query and are not stored
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) dst[ks] = load8<F32>(a.q, base + (int64_t)qi * a.sn + 16 * ks + 8 * g);
  };
  bf16x8 xf[KS];
  load_q(b_lo + w, xf);
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  __syncthreads();
  const float *b1 = &vecs[0], *b2 = &vecs[F], *zz = &vecs[2 * F];
  const lds_frag_ptr w1f = (lds_frag_ptr)&ops[0], w2f = (lds_frag_ptr)&ops[NOP];
  const lds_frag_ptr sth = (lds_frag_ptr)&ops[2 * NOP], stl = (lds_frag_ptr)&ops[3 * NOP];
  char *stage = stage_all + w * 32 * PITCH;

  for (int blk = b_lo + w; blk < b_hi; blk += 8) {
    f32x16 u[FB];
    {
      u32x4 h_hi[4][2], h_lo[4][2];
      mlp128_pipelined<ACT0, true>(xf, w1f, w2f, b1, b2, lane, g, a.act, h_hi, h_lo, u, [&]() { load_q(blk + 8, xf); });
    }
    if constexpr (P2) {
      // the paper's default degree: the upper half of the channels is squared
#pragma unroll
      for (int fb = FB / 2; fb < FB; ++fb)
#pragma unroll
        for (int x = 0; x < 16; ++x) u[fb][x] *= u[fb][x];
    } else if (a.P > 1) {
      // slice p = channel / (F / P) (0-based) gets p extra multiplications by the activation value
#pragma unroll
      for (int fb = 0; fb < FB; ++fb)
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const int extra = ((32 * fb + 8 * q) * a.P) / F;
          if (extra > 0) {
            const float t0 = u[fb][4 * q], t1 = u[fb][4 * q + 1], t2 = u[fb][4 * q + 2], t3 = u[fb][4 * q + 3];
            for (int i = 0; i < extra; ++i) {
              u[fb][4 * q] *= t0;
              u[fb][4 * q + 1] *= t1;
              u[fb][4 * q + 2] *= t2;
              u[fb][4 * q + 3] *= t3;
            }
          }
        }
    }
    // phi_q rounded to bf16: the B operand of the contraction (word i: channels crow(8 s + 2 i, g) and the next)
    u32x4 gb[FB][2];
#pragma unroll
    for (int fb = 0; fb < FB; ++fb)
#pragma unroll
      for (int s = 0; s < 2; ++s)
#pragma unroll
        for (int i = 0; i < 4; ++i) gb[fb][s][i] = pack_bf16(u[fb][8 * s + 2 * i], u[fb][8 * s + 2 * i + 1]);
    // n^T = S^T phi_q^T, two 32-channel row blocks at a time (two alternating accumulator chains), one 16-feature slice
    // (4 matrix instructions) per step; the fragments of the next step are requested behind the step's first matrix
    // instruction.  Under the first pair: the denominator, from the rounded features; under the second: the output
    // of the first.
    const int q_first = 32 * blk;
    f32x16 n[RB];
    float den = 0.f, inv = 0.f;
    auto den_slice = [&](int t, int half) {
      const int fb = t >> 1, s = t & 1;
      const f32x4 z4 = *reinterpret_cast<const f32x4 *>(zz + 32 * fb + 16 * s + 8 * half + 4 * g);
#pragma unroll
      for (int j = 0; j < 4; j += 2) {
        const unsigned pair = gb[fb][s][2 * half + j / 2];
        den = __builtin_fmaf(__uint_as_float(pair << 16), z4[j], den);
        den = __builtin_fmaf(__uint_as_float(pair & 0xffff0000u), z4[j + 1], den);
      }
    };
    // Output, 64 bytes of every row per pass: registers 4 x .. 4 x + 3 are channels 8 x + 4 g .. + 3 of query r.  The
    // staging area is the wave's own and a wave's LDS instructions execute in order, so the compiler only has to
    // keep the reads behind the writes (and the next pass's writes behind the reads).
    f32x4 out_piece[2];
    auto put = [&](int rb, int p, int xl) {
      const int x4 = p * (CPP / 8) + xl;
      const f32x4 y = {n[rb][4 * x4] * inv, n[rb][4 * x4 + 1] * inv, n[rb][4 * x4 + 2] * inv, n[rb][4 * x4 + 3] * inv};
      char *dst = stage + r * PITCH + (8 * xl + 4 * g) * ESZ;
      if constexpr (F32) *reinterpret_cast<f32x4 *>(dst) = y;
      else *reinterpret_cast<bf16x4 *>(dst) = __builtin_convertvector(y, bf16x4);
    };
    auto take = [&]() {
      asm volatile("" ::: "memory");
#pragma unroll
      for (int i = 0; i < 2; ++i) out_piece[i] = *reinterpret_cast<const f32x4 *>(stage + (16 * i + (lane >> 2)) * PITCH + (lane & 3) * 16);
      asm volatile("" ::: "memory");
    };
    auto store = [&](int rb, int p) {
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        const int row = 16 * i + (lane >> 2);
        char *dst = static_cast<char *>(a.out) + (base + (int64_t)(q_first + row) * a.sn + 32 * rb + CPP * p) * ESZ + (lane & 3) * 16;
        if (q_first + row < a.N) *reinterpret_cast<f32x4 *>(dst) = out_piece[i];
      }
    };
    auto store_part = [&](int rb, int x4) {                 // registers 4 x4 .. 4 x4 + 3 of row block rb
      a.lin[((((int64_t)bh * a.n_tb + blk) * RB + rb) * 4 + x4) * 64 + lane] =
          f32x4{n[rb][4 * x4], n[rb][4 * x4 + 1], n[rb][4 * x4 + 2], n[rb][4 * x4 + 3]};
    };
    constexpr int PASSES = 32 / CPP, SPP = 16 / PASSES;   // passes per row block, matrix-instruction slots per pass
    bf16x8 fa[2][2], fbuf[2][2];
    auto st_frags = [&](int rp, int t, bf16x8 (&dst)[2][2]) {
#pragma unroll
      for (int e = 0; e < 2; ++e) {
        dst[e][0] = frag_at(stl, (rp + e) * FB * 2 + t, lane);
        dst[e][1] = frag_at(sth, (rp + e) * FB * 2 + t, lane);
      }
    };
    st_frags(0, 0, fa);
#pragma unroll
    for (int rb = 0; rb < RB; ++rb)
#pragma unroll
      for (int x = 0; x < 16; ++x) n[rb][x] = 0.f;
    HA_FENCE();
#pragma unroll
    for (int rp = 0; rp < RB; rp += 2) {
#pragma unroll
      for (int t = 0; t < 2 * FB; ++t) {
        bf16x8 (&cur)[2][2] = (t & 1) ? fbuf : fa;
        bf16x8 (&nxt)[2][2] = (t & 1) ? fa : fbuf;
#pragma unroll
        for (int slot = 0; slot < 4; ++slot) {
          const int e = slot & 1, hi = slot >> 1;
          n[rp + e] = mfma32(cur[e][hi], __builtin_bit_cast(bf16x8, gb[t >> 1][t & 1]), n[rp + e]);
          if (slot == 0) {
            if (t + 1 < 2 * FB) st_frags(rp, t + 1, nxt);
            else if (rp + 2 < RB) st_frags(rp + 2, 0, nxt);
          }
          if (rp == 0) {
            if (slot >= 2) den_slice(t, slot - 2);
          } else if constexpr (PART) {
            if (t < 2) store_part(slot >> 1, 2 * (slot & 1) + t);       // the image of the first pair
          } else {
            const int c = t * 4 + slot, q = c / SPP, rb = q / PASSES, p = q % PASSES, at = c % SPP;
            if (at < CPP / 8) put(rb, p, at);
            else if (at == CPP / 8 + 2) take();
            else if (at == SPP - 2) store(rb, p);
          }
          HA_FENCE();
        }
      }
      if (rp == 0) {
        den = xhalf_sum(den);
        if (a.row_den && lane < 32 && q_first + lane < a.N) a.row_den[(int64_t)bh * a.N + q_first + lane] = den;
        if (PART && lane < 32 && q_first + lane < a.N) a.lin_e[(int64_t)bh * a.N + q_first + lane] = den;
        inv = 1.0f / den;
        HA_FENCE();
      }
    }
    if constexpr (PART) {
#pragma unroll
      for (int i = 0; i < 8; ++i) store_part(2 + (i >> 2), i & 3);
      continue;
    }
#pragma unroll
    for (int rb = 2; rb < RB; ++rb)
#pragma unroll
      for (int p = 0; p < PASSES; ++p) {
#pragma unroll
        for (int xl = 0; xl < CPP / 8; ++xl) put(rb, p, xl);
        take();
        store(rb, p);
      }
  }
}

hipError_t launch_linear_query(const Plan &pl, const void *q, const ha_feature_map &phi_q, void *out, float *row_den, void *ws,
                               hipStream_t st) {
  char *wsb = static_cast<char *>(ws);
  LinearArgs a;
  a.q = q;
  a.out = out;
  a.row_den = row_den;
  a.w1f = reinterpret_cast<bf16x8 *>(wsb + pl.off_w1q);
  a.w2f = reinterpret_cast<bf16x8 *>(wsb + pl.off_w2q);
  a.b1 = phi_q.b1;
  a.b2 = phi_q.b2;
  a.st_hi = reinterpret_cast<bf16x8 *>(wsb + pl.off_sthi);
  a.st_lo = reinterpret_cast<bf16x8 *>(wsb + pl.off_stlo);
  a.z = reinterpret_cast<float *>(wsb + pl.off_z);
  a.H = pl.H; a.N = pl.N; a.P = pl.P; a.act = pl.act_q;
  a.sb = pl.sb; a.sh = pl.sh; a.sn = pl.sn;
  const bool part = pl.split_linear;
  a.lin = part ? reinterpret_cast<f32x4 *>(wsb + pl.off_lin) : nullptr;
  a.lin_e = part ? reinterpret_cast<float *>(wsb + pl.off_e) : nullptr;
  a.n_tb = pl.n_tb;
  // one workgroup per CU in a single round; short sequences spread over as many of them as they have blocks
  const int nb = (pl.N + 31) / 32, room = 256 / (pl.B * pl.H) > 0 ? 256 / (pl.B * pl.H) : 1;
  a.per_bh = nb < room ? nb : room;
  a.total = a.per_bh * pl.B * pl.H;
  const int grid = (a.total + 7) / 8 * 8;
#define HA_LINEAR(F32, PART) \
  do { \
    if (pl.act_q != HA_ACT_SOFTMAX) linear_query_kernel<F32, false, false, PART><<<grid, 512, 0, st>>>(a); \
    else if (pl.P == 2) linear_query_kernel<F32, true, true, PART><<<grid, 512, 0, st>>>(a); \
    else linear_query_kernel<F32, true, false, PART><<<grid, 512, 0, st>>>(a); \
  } while (0)
  if (part) { if (pl.f32) HA_LINEAR(true, true); else HA_LINEAR(false, true); }
  else { if (pl.f32) HA_LINEAR(true, false); else HA_LINEAR(false, false); }
#undef HA_LINEAR
  return hipGetLastError();
}

}  // namespace ha
