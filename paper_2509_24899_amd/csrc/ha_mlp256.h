// Pieces of the feature map phi of Sec. 3.2 for the widths 128 -> 256 -> 256 on one 32-token column block, shared by the state
// pass and the query side.  gfx950 only.
//
// A token's 256 pre-activations are eight accumulator tiles; the hidden layer is walked in blocks of 32 units, each formed
// (8 matrix instructions), split into hi + lo and contracted into all eight tiles (32 instructions).  The operands of a step form a
// 24 KiB slab: the 8 fragments of a block's rows of W1, then for every 32-channel output tile the two of the block's columns of W2.
// Two forms:
//   query side (mlp256_hidden_block)     a block is formed at the head of its own step and is all that is held; its slab brings
//                                        its own rows of W1
//   state pass (hidden_block_products)   the next block is formed under the current one's products, two blocks are held; a slab
//                                        brings the rows of W1 of the block after its own
#pragma once
#include "ha_mlp128.h"

namespace ha {

constexpr int kSlabChunks = 8 + 2 * 8;                    // 1 KiB chunks of a weight slab
// Chunk c of the slab of hidden block hb, from one head's prepared fragments (W1 natural, W2 chained order).
static __device__ __forceinline__ const bf16x8 *slab_chunk(const bf16x8 *w1f, const bf16x8 *w2f, int hb, int c) {
  return c < 8 ? w1f + (hb * 8 + c) * 64 : w2f + ((((c - 8) >> 1) * 8 + hb) * 2 + ((c - 8) & 1)) * 64;
}

// 32 consecutive values (LDS) as one column of a C tile: four 16-byte reads, no vector instruction.
static __device__ __forceinline__ f32x16 column_tile(const float *b, int blk, int g) {
  const f32x4 *src = reinterpret_cast<const f32x4 *>(b + 32 * blk + 4 * g);
  const f32x8 lo = __builtin_shufflevector(src[0], src[2], 0, 1, 2, 3, 4, 5, 6, 7);
  const f32x8 hi = __builtin_shufflevector(src[4], src[6], 0, 1, 2, 3, 4, 5, 6, 7);
  return __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7, 8, 9, 10, 11, 12, 13, 14, 15);
}

// Registers x, x + 1 of a finished hidden tile -> ReLU -> hi + lo.
static __device__ __forceinline__ void split2(const f32x16 &hh, int x, u32x4 (&hi)[2], u32x4 (&lo)[2]) {
  const float v0 = relu(hh[x]), v1 = relu(hh[x + 1]);
  const unsigned p = pack_bf16(v0, v1);
  hi[x >> 3][(x & 7) >> 1] = p;
  lo[x >> 3][(x & 7) >> 1] = pack_bf16(v0 - __uint_as_float(p << 16), v1 - __uint_as_float(p & 0xffff0000u));
}

// ReLU of a finished hidden tile as hi + lo bf16 pairs: the B operands of the next product.
static __device__ __forceinline__ void relu_hi_lo(const f32x16 &t, u32x4 (&hi)[2], u32x4 (&lo)[2]) {
#pragma unroll
  for (int x = 0; x < 16; x += 2) split2(t, x, hi, lo);
}

// relu(W1[block, :] x + b1[block]) of hidden block hb from the head of its slab.
static __device__ __forceinline__ void hidden_block(lds_frag_ptr sl, const float *b1, int hb, const bf16x8 (&xf)[8], int lane, int g,
                                                    u32x4 (&h_hi)[2], u32x4 (&h_lo)[2]) {
  f32x16 hh = column_tile(b1, hb, g);
#pragma unroll
  for (int ks = 0; ks < 8; ++ks) hh = mfma32(frag_at(sl, ks, lane), xf[ks], hh);
  relu_hi_lo(hh, h_hi, h_lo);
}

// u += W[:, block] h of the block's 32 inputs for NT output tiles; wsl: two fragments per tile.
template <int NT>
static __device__ __forceinline__ void hidden_to_outputs(lds_frag_ptr wsl, bf16x8 hi0, bf16x8 hi1, bf16x8 lo0, bf16x8 lo1, int lane,
                                                         f32x16 (&u)[NT]) {
#pragma unroll
  for (int s = 0; s < 2; ++s) {
    const bf16x8 hi8 = s ? hi1 : hi0, lo8 = s ? lo1 : lo0;
#pragma unroll
    for (int fb = 0; fb < NT; fb += 2) {
      const bf16x8 wa = frag_at(wsl, 2 * fb + s, lane), wb = frag_at(wsl, 2 * (fb + 1) + s, lane);
      u[fb] = mfma32(wa, lo8, u[fb]);
      u[fb + 1] = mfma32(wb, lo8, u[fb + 1]);
      u[fb] = mfma32(wa, hi8, u[fb]);
      u[fb + 1] = mfma32(wb, hi8, u[fb + 1]);
    }
  }
}

// u += W2[:, block] relu(W1[block, :] x + b1[block]) from the block's slab in LDS.
static __device__ __forceinline__ void mlp256_hidden_block(lds_frag_ptr sl, const float *b1, int hb, const bf16x8 (&xf)[8],
                                                           int lane, int g, f32x16 (&u)[8]) {
  u32x4 h_hi[2], h_lo[2];
  hidden_block(sl, b1, hb, xf, lane, g, h_hi, h_lo);
  hidden_to_outputs<8>(sl + 8 * 64, __builtin_bit_cast(bf16x8, h_hi[0]), __builtin_bit_cast(bf16x8, h_hi[1]),
                       __builtin_bit_cast(bf16x8, h_lo[0]), __builtin_bit_cast(bf16x8, h_lo[1]), lane, u);
}

// The products of a hidden block come in 8 groups of four: group gi = (half s, output tiles fb, fb + 1).
static __device__ __forceinline__ void read_group256(lds_frag_ptr wsl, int gi, int lane, bf16x8 (&fr)[2][2]) {
  const int s = gi >> 2, fb = 2 * (gi & 3);
  fr[gi & 1][0] = frag_at(wsl, 2 * fb + s, lane);
  fr[gi & 1][1] = frag_at(wsl, 2 * fb + 2 + s, lane);
}
// u += W2[:, block] h for the hidden block in h_hi, h_lo, and, NEXT, under it the next one, nb: its matrix instructions in the
// first half, its ReLU and hi + lo split in the second; on return h_hi, h_lo hold it.  wsl: the 16 fragments of the block's columns
// of W2, of which group 0 has been read into fr; w1_next: the 8 of the next block's rows of W1.
// (Formed at the head of its own block the hidden block is eight matrix instructions in series with nothing beside them.)
template <bool NEXT>
static __device__ __forceinline__ void hidden_block_products(lds_frag_ptr wsl, lds_frag_ptr w1_next, const float *b1,
                                                             int nb, const bf16x8 (&xf)[8], int lane, int g, bf16x8 (&fr)[2][2],
                                                             u32x4 (&h_hi)[2], u32x4 (&h_lo)[2], f32x16 (&u)[8]) {
  f32x16 hh;
  bf16x8 wl[2][2];
  u32x4 n_hi[2], n_lo[2];
  if constexpr (NEXT) {
    hh = column_tile(b1, nb, g);
    wl[0][0] = frag_at(w1_next, 0, lane);
    wl[0][1] = frag_at(w1_next, 1, lane);
  }
#pragma unroll
  for (int gi = 0; gi < 8; ++gi) {
    if (gi < 7) read_group256(wsl, gi + 1, lane, fr);
    if (NEXT && gi < 3) {
      wl[(gi + 1) & 1][0] = frag_at(w1_next, 2 * gi + 2, lane);
      wl[(gi + 1) & 1][1] = frag_at(w1_next, 2 * gi + 3, lane);
    }
    HA_FENCE();
    const int s = gi >> 2, fb = 2 * (gi & 3);
    const bf16x8 hi8 = __builtin_bit_cast(bf16x8, h_hi[s]), lo8 = __builtin_bit_cast(bf16x8, h_lo[s]);
    u[fb] = mfma32(fr[gi & 1][0], lo8, u[fb]);
    u[fb + 1] = mfma32(fr[gi & 1][1], lo8, u[fb + 1]);
    u[fb] = mfma32(fr[gi & 1][0], hi8, u[fb]);
    u[fb + 1] = mfma32(fr[gi & 1][1], hi8, u[fb + 1]);
    if constexpr (NEXT) {
      if (gi < 4) {
        hh = mfma32(wl[gi & 1][0], xf[2 * gi], hh);
        hh = mfma32(wl[gi & 1][1], xf[2 * gi + 1], hh);
      } else {
        split2(hh, 4 * (gi - 4), n_hi, n_lo);
        split2(hh, 4 * (gi - 4) + 2, n_hi, n_lo);
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
          __builtin_amdgcn_sched_group_barrier(0x002, 4, 0);
        }
      }
    }
    HA_FENCE();
  }
  if constexpr (NEXT) {
#pragma unroll
    for (int s = 0; s < 2; ++s) {
      h_hi[s] = n_hi[s];
      h_lo[s] = n_lo[s];
    }
  }
}

// The output stage in place: positive activation over all channels, slice powers.  ACT0: softmax over the channels; otherwise
// `act` picks exp (1) or ReLU.  P2: the degree is 2, the paper's default.  Tile by tile against the running maximum, the
// exponentials rounded to bf16 as they are formed and phi once more behind the powers: value for value what the tile-wise form
// (feature_layer2_phi_tiles, feature_phi_finish) does, which the variants' epilogue uses.
template <bool ACT0, bool P2>
static __device__ __forceinline__ void phi256_output(f32x16 (&u)[8], int act, int P) {
  float factor[8];
  if constexpr (ACT0) {
    float m_run = kMaxFloor, sum = 0.f;
#pragma unroll
    for (int fb = 0; fb < 8; ++fb) {
      float t = u[fb][0];
#pragma unroll
      for (int x = 1; x < 16; ++x) t = fmaxf(t, u[fb][x]);
      const float m_new = fmaxf(m_run, xhalf_max(t));
      sum *= fast_exp2((m_run - m_new) * kLog2e);         // (the sum is 0 on the first tile)
      const float off = -m_new * kLog2e;
#pragma unroll
      for (int x = 0; x < 16; x += 2) {
        const float e0 = fast_exp2(__builtin_fmaf(u[fb][x], kLog2e, off)), e1 = fast_exp2(__builtin_fmaf(u[fb][x + 1], kLog2e, off));
        sum += e0;
        sum += e1;
        const unsigned p = pack_bf16(e0, e1);
        u[fb][x] = __uint_as_float(p << 16);
        u[fb][x + 1] = __uint_as_float(p & 0xffff0000u);
      }
      factor[fb] = m_run = m_new;
    }
    const float inv = 1.0f / xhalf_sum(sum);
#pragma unroll
    for (int fb = 0; fb < 8; ++fb) factor[fb] = fast_exp2((factor[fb] - m_run) * kLog2e) * inv;
  } else {
#pragma unroll
    for (int fb = 0; fb < 8; ++fb)
#pragma unroll
      for (int x = 0; x < 16; ++x) u[fb][x] = act == 1 ? fast_exp2(u[fb][x] * kLog2e) : relu(u[fb][x]);
  }
#pragma unroll
  for (int fb = 0; fb < 8; ++fb) {
    if constexpr (ACT0) {
#pragma unroll
      for (int x = 0; x < 16; ++x) u[fb][x] *= factor[fb];
    }
    if constexpr (P2) {                                   // the upper half of the channels is squared
      if (fb >= 4)
#pragma unroll
        for (int x = 0; x < 16; ++x) u[fb][x] *= u[fb][x];
    } else {
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int extra = ((32 * fb + 8 * q) * P) / 256;  // slice = power - 1 in 0 .. 7; wave-uniform
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
}

}  // namespace ha
