// Layers of the feature maps that go layer by layer through HBM (ha_wide.hip), as one streaming kernel.  gfx950 only.
//
// One workgroup, 8 waves of 32 tokens, walks a contiguous run of work items (tile of 256 tokens, block of 32 NT output
// channels).  A wave's accumulators are the NT output tiles of its tokens; the contraction runs over the input width in
// blocks of 32, each of which is
//   from x      formed on the spot: relu(W1 x + b1) of 32 hidden units (8 matrix instructions), split into hi + lo, so that
//               the first hidden layer never visits HBM (its 8 instructions per block are repeated for every block of output
//               channels: a quarter of the 32 that consume it, against 4 bytes per unit and token written and read back), or
//   from HBM    fetched as the hi + lo register images the previous layer left, three blocks ahead.
// The weights of a block (its rows of W1, its columns of the layer's matrix) are one slab of an LDS ring that all waves
// share; requests run ahead across items, one barrier per block.  A slab is in place a block before its turn, so that under the
// products of a block the next block's first fragments are read and (from x) the next hidden block is formed: formed at the head
// of its own block, as eight products in series each behind an LDS read of its own, it left the matrix cores idle in both waves of a
// SIMD at once (57 % busy, now 64 %; from HBM 50 %, now 58 - 64 %).  From HBM the output blocks of a tile go to neighbouring workgroups of an XCD at the same
// time, so that its image is fetched once: one after the other in one workgroup it was fetched three times (3.8 GB, now 1.5 GB).
//
// Outputs leave in a burst per item, and slabs requested behind them are not known to have landed before they have reached memory
// (loads and stores retire in order): the ring is as long as LDS and the contraction allow, the input's next blocks are requested
// ahead of the outputs.
//
// Bound: matrix cores at the power limit: 1.25 - 1.3 PFLOP/s of matrix instructions in both forms (steady slabs take 1.17 times their
// matrix instructions' cycles; clock 1.8 - 1.9 GHz), where a large library product of the same type reaches 1.3.  Measured with the
// 768-wide three-layer maps at 480p / 81 frames, 12 heads, R = 8, keys and queries, before and after on one box: from x 856 and 925 us
// with the hidden block at the head of its own block, 806 and 891 us here; from HBM 777 and 892 us with a wait for all loads every
// fourth block and the image fetched three times, 632 and 703 us here.  Two slabs per barrier took 9.4 k cycles instead of 9.7 k for
// four slabs and no less time.  The 256-wide maps' two layers ahead of a backward pass: 111 + 174 us as passes of their own, 185 us
// here (queries).
#include "ha_mlp256.h"
#include "ha_plan.h"

namespace ha {

struct WideMlpArgs {
  const void *x;                 // from x: q or k (io dtype, strided)
  const bf16x8 *in_hi, *in_lo;   // from HBM: the previous layer's images, width K
  const bf16x8 *w1f, *wf;        // fragments, all heads: W1 (natural order), this layer's matrix [NOUT x K] (chained)
  const float *b1, *bias;        // [H][K], [H][NOUT], or null
  bf16x8 *h_hi;                  // from x: the hidden layer's bf16 image, if somebody needs it (or null)
  bf16x8 *out_hi, *out_lo;       // hidden layer out
  f32x4 *out_u;                  // last layer: fp32 pre-activations
  float *out_stat;               // last layer: [bh][tb][128-channel block][2][64] maximum and sum of exponentials
  int H, K, NOUT, n_tok, n_tb, R, G;
  int ob_first, n_ob;            // first output tile, blocks of NT tiles
  int n_tiles;                   // 256-token tiles per (batch, head)
  int first, total;              // items of this launch
  int64_t sb, sh, sn;
};

// Maximum and sum over the 32 lanes of a half wave, in every one of them.
template <int CTRL>
static __device__ __forceinline__ float dpp(float x) {
  return __uint_as_float(__builtin_amdgcn_update_dpp(0, __float_as_uint(x), CTRL, 0xf, 0xf, true));
}
static __device__ __forceinline__ float half_max(float x) {
  x = fmaxf(x, dpp<0xB1>(x));                      // lane ^ 1, lane ^ 2, then mirrored eights and sixteens
  x = fmaxf(x, dpp<0x4E>(x));
  x = fmaxf(x, dpp<0x141>(x));
  x = fmaxf(x, dpp<0x140>(x));
  const u32x2 p = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return fmaxf(__uint_as_float(p[0]), __uint_as_float(p[1]));
}
static __device__ __forceinline__ float half_sum(float x) {
  x += dpp<0xB1>(x);
  x += dpp<0x4E>(x);
  x += dpp<0x141>(x);
  x += dpp<0x140>(x);
  const u32x2 p = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return __uint_as_float(p[0]) + __uint_as_float(p[1]);
}

// SRC: 0 from x in bf16, 1 from x in fp32, 2 from HBM.  OUT: 0 relu, hi + lo bf16 (a hidden layer); 1 fp32 pre-activations (the last
// layer), a token per lane; 2 the same with a channel per lane and the tokens in the registers, for the state pass, whose
// contraction over the tokens takes them as they are: the operands of every product change places, nothing else.
// NBUF: slabs in the ring, at most K / 32 + 1.
template <int NT, int SRC, int OUT, int NBUF>
__global__ __launch_bounds__(512, 2) void wide_mlp_kernel(WideMlpArgs a) {
  constexpr bool X = SRC != 2, LAST = OUT != 0, TR = OUT == 2;
  constexpr int D = 128, KS = D / 16, NW = 8;
  constexpr int CH = (X ? KS : 0) + 2 * NT, PW = CH / NW, SLOT = CH * 64;      // 1 KiB chunks per slab, per wave
  constexpr int WMAX = 768;
  static_assert(CH % NW == 0 && KS == NW, "slabs are dealt evenly, the first chunk of a wave from W1");
  __shared__ bf16x8 ring[NBUF * SLOT];
  __shared__ __align__(16) float vecs[(X ? WMAX : 0) + WMAX];                  // b1, bias of the whole layer
  const int tid = threadIdx.x, lane = tid & 63, r = lane & 31, g = lane >> 5;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  // Items of this workgroup: from x a contiguous run, so that a tile's rows and first hidden block serve all its output blocks;
  // from HBM the items of its XCD in turn, so that neighbouring workgroups read a tile's image at the same time and it leaves
  // HBM (or the cache in front of it) once and not once per output block.
  const int per_xcd = gridDim.x >> 3, xcd = blockIdx.x & 7, in_xcd = blockIdx.x >> 3;   // the grid is a multiple of 8
  const int u_lo = X ? xcd * per_xcd + in_xcd : xcd, u_n = X ? gridDim.x : 8, stride = X ? 1 : per_xcd;
  const int i_lo = a.first + (int)((int64_t)u_lo * a.total / u_n) + (X ? 0 : in_xcd), i_hi = a.first + (int)((int64_t)(u_lo + 1) * a.total / u_n);
  if (i_lo >= i_hi) return;
  const int KB = a.K / 32, OB = a.NOUT / 32;                                   // KB: a multiple of 4
  const int per_head = a.n_tiles * a.n_ob;
  const LinearMap lmap(a.R, a.G);

  struct Item {
    int bh, tb, ob0;                                                           // tb: this wave's 32-token block
    const bf16x8 *w1, *wm;                                                     // this wave's chunks of slab 0
    int64_t image;                                                             // from HBM: block 0 of the input's image
  };
  auto item_of = [&](int i) {
    Item it;
    it.bh = i / per_head;
    const int rem = i - it.bh * per_head, tile = rem / a.n_ob, h = it.bh % a.H;
    it.tb = tile * NW + w;
    it.ob0 = a.ob_first + (rem - tile * a.n_ob) * NT;
    // chunk NW i + w of a slab is (X) chunk w of the block's W1 for i = 0, then fragment w % 2 of output tile 4 i' + w / 2
    it.w1 = X ? a.w1f + (int64_t)h * (a.K * D / 8) + w * 64 : nullptr;
    it.wm = a.wf + (int64_t)h * ((int64_t)a.NOUT * a.K / 8) + ((int64_t)(it.ob0 + (w >> 1)) * KB * 2 + (w & 1)) * 64;
    it.image = ((int64_t)it.bh * a.n_tb + min(it.tb, a.n_tb - 1)) * KB * 128;
    return it;
  };
  const unsigned lane_off = lane * 16;
  const unsigned ring_w = (unsigned)(uintptr_t)(__attribute__((address_space(3))) void *)(&ring[0]) + w * 1024;
  auto request = [&](const Item &it, int kb, int slot) {
    const bf16x8 *wm = it.wm + kb * 128;
#pragma unroll
    for (int i = 0; i < PW; ++i) {
      const bf16x8 *gp = X && i == 0 ? it.w1 + kb * (KS * 64) : wm + (int64_t)(i - (X ? 1 : 0)) * (4 * 128) * KB;
      const unsigned l = __builtin_amdgcn_readfirstlane(ring_w + (slot * SLOT + i * NW * 64) * 16);
      asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2" ::"s"(l), "v"(lane_off), "s"(gp) : "memory");
    }
  };
  Item cur = item_of(i_lo), nxt = cur;
  int slot = 0;                                    // slot of the current slab
  bool stored = false;                             // this wave wrote its outputs at the end of the item before
  // Barrier ahead of slab kb: this wave's shares of slabs kb and kb + 1 have landed and so have everybody's, and everybody is
  // done with slab kb - 1, whose slot takes the request NBUF - 1 slabs ahead.  (Slab kb itself was there a barrier ago, so that
  // its first fragments are read ahead of this barrier, under the products of slab kb - 1; all reads of slab kb - 1 have been
  // used by then.)  Newer than the request of slab kb + 1 are at least NBUF - 3 requests (and from HBM NBUF - 2 groups of four
  // image loads), and, where that request came before this wave's outputs, those 4 NT stores (loads and stores retire in order, so
  // that the ring's length is what the outputs have to reach memory in).  The counter ends at 63 operations, so that a wait for 63
  // is none: where more than 62 are newer (NT = 8 with nine slabs: 72), the wait is for all but 62.  The slabs requested ahead of the
  // first item are waited for together.
  constexpr int FLY = (NBUF - 3) * PW + (X ? 0 : (NBUF - 2) * 4), FLY_OUT = FLY + 4 * NT < 62 ? FLY + 4 * NT : 62;
  static_assert(FLY <= 62, "a wait that the counter can hold");
  auto advance = [&](int kb) {
    if (stored && kb < NBUF - 2) asm volatile("s_waitcnt vmcnt(%0)\n\ts_barrier" ::"n"(FLY_OUT) : "memory");
    else asm volatile("s_waitcnt vmcnt(%0)\n\ts_barrier" ::"n"(FLY) : "memory");
  };
  auto refill = [&](int kb) {                      // (behind a slab's first products, under which its scalar instructions pass)
    const int s = kb + NBUF - 1;
    request(s < KB ? cur : nxt, s < KB ? s : s - KB, slot == 0 ? NBUF - 1 : slot - 1);   // (past the last item: a slab nobody reads)
  };
  auto slab = [&](int s) { return (lds_frag_ptr)&ring[s * SLOT]; };
  auto next_slot = [&]() { return slot + 1 == NBUF ? 0 : slot + 1; };

  bf16x8 xf[X ? KS : 1];
  auto load_x = [&](const Item &it) {
    const int h = it.bh % a.H;
    const int64_t base = (int64_t)(it.bh / a.H) * a.sb + (int64_t)h * a.sh;
    const int tok = lmap.token(min(32 * it.tb + r, a.n_tok - 1));              // rows past the end repeat the last token
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) xf[ks] = load8<SRC == 1>(a.x, base + (int64_t)tok * a.sn + 16 * ks + 8 * g);
  };
  bf16x8 im_hi[X ? 1 : 4][2], im_lo[X ? 1 : 4][2];                             // input blocks kb .. kb + 3, buffer kb % 4
  auto load_image = [&](const Item &it, int kb, bf16x8 (&hi)[2], bf16x8 (&lo)[2]) {
    const bf16x8 *ph = a.in_hi + it.image + kb * 128, *pl = a.in_lo + it.image + kb * 128;
#pragma unroll
    for (int s = 0; s < 2; ++s) {
      hi[s] = ph[s * 64 + lane];
      lo[s] = pl[s * 64 + lane];
    }
  };
#pragma unroll
  for (int s = 0; s < NBUF - 1; ++s) request(cur, s, s);                       // (KB >= NBUF - 1)
  if constexpr (!X) {
    // in this order: the compiler counts the loads that may be in flight at the head of the loop over all ways into it
#pragma unroll
    for (int s = 0; s < 4; ++s) {
      load_image(cur, s, im_hi[s], im_lo[s]);
      HA_FENCE();
    }
  }
  const float *b1 = &vecs[0], *bias = &vecs[X ? WMAX : 0];

  // The products of a slab: NT groups of four, group gi = (half s, output tiles fb, fb + 1); the fragments of a group are read
  // LA groups ahead, those of the next slab's first groups included.
  constexpr int LA = X ? 1 : 2, NF = 2 * LA;
  static_assert(NT % NF == 0, "the fragment buffers rotate whole within a slab");
  bf16x8 fr[NF][2];
  constexpr int W0 = X ? KS : 0;                                               // first weight chunk behind W1
  auto read_group = [&](lds_frag_ptr sl, int gi) {
    const int s = gi / (NT / 2), fb = 2 * (gi % (NT / 2));
    fr[gi % NF][0] = frag_at(sl, W0 + 2 * fb + s, lane);
    fr[gi % NF][1] = frag_at(sl, W0 + 2 * fb + 2 + s, lane);
  };
  f32x16 acc[NT];
  auto products = [&](int gi, bf16x8 hi8, bf16x8 lo8) {
    const int fb = 2 * (gi % (NT / 2));
    auto mul = [](bf16x8 wgt, bf16x8 h, f32x16 c) { return TR ? mfma32(h, wgt, c) : mfma32(wgt, h, c); };
    acc[fb] = mul(fr[gi % NF][0], lo8, acc[fb]);
    acc[fb + 1] = mul(fr[gi % NF][1], lo8, acc[fb + 1]);
    acc[fb] = mul(fr[gi % NF][0], hi8, acc[fb]);
    acc[fb + 1] = mul(fr[gi % NF][1], hi8, acc[fb + 1]);
  };
  u32x4 h_hi[2], h_lo[2];                                                      // from x: the hidden block of the current slab
  auto hop = [](const u32x4 &t) { return __builtin_bit_cast(bf16x8, t); };

  int bh_vecs = -1, x_bh = -1, x_tb = -1;
  for (int i = i_lo; i < i_hi; i += stride) {
    nxt = item_of(i + stride < i_hi ? i + stride : i);
    const bool new_x = X && (cur.bh != x_bh || cur.tb != x_tb);                // workgroup-uniform
    if (cur.bh != bh_vecs) {                       // workgroup-uniform: the first item, or the head changes
      const int h = cur.bh % a.H;
      __syncthreads();                             // every wave is done with the previous head's biases
      if constexpr (X)
        for (int j = tid; j < a.K; j += 512) vecs[j] = a.b1 ? a.b1[(int64_t)h * a.K + j] : 0.f;
      for (int j = tid; j < a.NOUT; j += 512) vecs[(X ? WMAX : 0) + j] = a.bias ? a.bias[(int64_t)h * a.NOUT + j] : 0.f;
      bh_vecs = cur.bh;
      __syncthreads();
    }
    if (i == i_lo) {
      // slab 0 is in place (from the second item on the barrier of the slab before has seen to it)
      asm volatile("s_waitcnt vmcnt(0)\n\ts_barrier" ::: "memory");
#pragma unroll
      for (int gi = 0; gi < LA; ++gi) read_group(slab(slot), gi);
    }
    const bool live = cur.tb < a.n_tb;             // idle waves keep staging and synchronising
#pragma unroll
    for (int j = 0; j < NT; ++j) {
      if constexpr (TR) {
        float b = bias[32 * (cur.ob0 + j) + r];
#pragma unroll
        for (int v = 0; v < 16; ++v) {
          asm volatile("" : "+v"(b));           // (sixteen copies: known to be one value, the tile was kept twice, in scratch)
          acc[j][v] = b;
        }
      } else {
        acc[j] = column_tile(bias, cur.ob0 + j, g);
      }
    }
    if constexpr (X) {
      if (new_x) {                                 // the first hidden block of a tile; the others are formed on the way
        load_x(cur);
        hidden_block(slab(slot), b1, 0, xf, lane, g, h_hi, h_lo);
        x_bh = cur.bh;
        x_tb = cur.tb;
      }
      const bool keep = a.h_hi && cur.ob0 == 0 && live;
      constexpr int HALF = NT / 2, PER = KS / HALF;                            // groups of either half, matrix instructions of W1 per group
#pragma unroll 1
      for (int kb = 0; kb < KB; ++kb) {
        advance(kb);
        if (keep) {
          const int64_t at = (((int64_t)cur.bh * a.n_tb + cur.tb) * KB + kb) * 128 + lane;
#pragma unroll
          for (int s = 0; s < 2; ++s) a.h_hi[at + s * 64] = hop(h_hi[s]);
        }
        // Under the products of this block: the next hidden block, its matrix instructions in the first half, its ReLU and
        // hi + lo split in the second.  (Behind the last block: block 0 once more, for the tile's next output channels.)
        const lds_frag_ptr sl = slab(slot), sn = slab(next_slot());
        f32x16 hh = column_tile(b1, kb + 1 < KB ? kb + 1 : 0, g);
        bf16x8 wl[2][PER];
        u32x4 n_hi[2], n_lo[2];
#pragma unroll
        for (int q = 0; q < PER; ++q) wl[0][q] = frag_at(sn, q, lane);
#pragma unroll
        for (int gi = 0; gi < NT; ++gi) {
          read_group(gi + LA < NT ? sl : sn, (gi + LA) % NT);
          if (gi + 1 < HALF) {
#pragma unroll
            for (int q = 0; q < PER; ++q) wl[(gi + 1) & 1][q] = frag_at(sn, (gi + 1) * PER + q, lane);
          }
          HA_FENCE();
          products(gi, hop(h_hi[gi / HALF]), hop(h_lo[gi / HALF]));
          if (gi == 0) {
            HA_FENCE();
            refill(kb);
            HA_FENCE();
          }
          if (gi < HALF) {
#pragma unroll
            for (int q = 0; q < PER; ++q) hh = mfma32(wl[gi & 1][q], xf[gi * PER + q], hh);
          } else {
#pragma unroll
            for (int q = 0; q < PER; ++q) split2(hh, 2 * ((gi - HALF) * PER + q), n_hi, n_lo);
#pragma unroll
            for (int q = 0; q < 4; ++q) {
              __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
              __builtin_amdgcn_sched_group_barrier(0x002, 2 * PER, 0);
            }
          }
          HA_FENCE();
        }
#pragma unroll
        for (int s = 0; s < 2; ++s) {
          h_hi[s] = n_hi[s];
          h_lo[s] = n_lo[s];
        }
        slot = next_slot();
      }
    } else {
#pragma unroll 1
      for (int kb = 0; kb < KB; kb += 4) {
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          advance(kb + q);
          const lds_frag_ptr sl = slab(slot), sn = slab(next_slot());
#pragma unroll
          for (int gi = 0; gi < NT; ++gi) {
            read_group(gi + LA < NT ? sl : sn, (gi + LA) % NT);
            HA_FENCE();
            products(gi, im_hi[q][gi / (NT / 2)], im_lo[q][gi / (NT / 2)]);
            HA_FENCE();
            if (gi == 0) {
              refill(kb + q);
              HA_FENCE();
            }
          }
          const int s = kb + q + 4;                // (ahead of this wave's outputs, where they follow)
          load_image(s < KB ? cur : nxt, s < KB ? s : s - KB, im_hi[q], im_lo[q]);
          HA_FENCE();
          slot = next_slot();
        }
      }
    }
    stored = live;
    if (live) {
      const int64_t blk0 = ((int64_t)cur.bh * a.n_tb + cur.tb) * OB + cur.ob0;
      if constexpr (LAST) {
#pragma unroll
        for (int j = 0; j < NT; ++j)
#pragma unroll
          for (int x4 = 0; x4 < 4; ++x4)
            a.out_u[((blk0 + j) * 4 + x4) * 64 + lane] = f32x4{acc[j][4 * x4], acc[j][4 * x4 + 1], acc[j][4 * x4 + 2], acc[j][4 * x4 + 3]};
        if constexpr (TR) {
          // per token (register v of half g: token crow(v, g) of the block) the maximum over this item's channels and the sum of exponentials
          // against it, in the statistics of the first 128 of them; a second 128 hold nothing more
          f32x4 m = {0.f, 0.f, 0.f, 0.f}, sum = m;           // lane r < 4 keeps registers 4 r .. 4 r + 3: tokens 8 r + 4 g .. + 3
#pragma unroll
          for (int v = 0; v < 16; ++v) {
            float t = acc[0][v];
#pragma unroll
            for (int j = 1; j < NT; ++j) t = fmaxf(t, acc[j][v]);
            const float mv = __builtin_fmaxf(half_max(t), kMaxFloor), off = -mv * kLog2e;
            t = 0.f;
#pragma unroll
            for (int j = 0; j < NT; ++j) t += fast_exp2(__builtin_fmaf(acc[j][v], kLog2e, off));
            const float sv = half_sum(t);
            m[v & 3] = r == v / 4 ? mv : m[v & 3];
            sum[v & 3] = r == v / 4 ? sv : sum[v & 3];
            if (v % 2) HA_FENCE();                           // (two chains at a time: the registers are full)
          }
          if (r < 4) {
            float *st = a.out_stat + ((((int64_t)cur.bh * a.n_tb + cur.tb) * (OB / 4) + cur.ob0 / 4) * 2) * 64 + 8 * r + 4 * g;
            *reinterpret_cast<f32x4 *>(st) = m;
            *reinterpret_cast<f32x4 *>(st + 64) = sum;
            if constexpr (NT == 8) {
              *reinterpret_cast<f32x4 *>(st + 128) = f32x4{-INFINITY, -INFINITY, -INFINITY, -INFINITY};
              *reinterpret_cast<f32x4 *>(st + 192) = f32x4{0.f, 0.f, 0.f, 0.f};
            }
          }
        } else {
          // per token and 128 channels: their maximum and the sum of exponentials against it, so that the output stage can
          // form the softmax over all channels with a single sweep over the pre-activations
#pragma unroll
          for (int j0 = 0; j0 < NT; j0 += 4) {
            float m = acc[j0][0];
#pragma unroll
            for (int j = j0; j < j0 + 4; ++j)
#pragma unroll
              for (int v = 0; v < 16; v += 2) m = __builtin_fmaxf(__builtin_fmaxf(m, acc[j][v]), acc[j][v + 1]);
            m = __builtin_fmaxf(xhalf_max(m), kMaxFloor);
            const float off = -m * kLog2e;
            float sum = 0.f;
#pragma unroll
            for (int j = j0; j < j0 + 4; ++j)
#pragma unroll
              for (int v = 0; v < 16; ++v) sum += fast_exp2(__builtin_fmaf(acc[j][v], kLog2e, off));
            sum = xhalf_sum(sum);
            float *st = a.out_stat + ((((int64_t)cur.bh * a.n_tb + cur.tb) * (OB / 4) + (cur.ob0 + j0) / 4) * 2) * 64 + lane;
            st[0] = m;
            st[64] = sum;
          }
        }
      } else {
#pragma unroll
        for (int j = 0; j < NT; ++j) {
          u32x4 hi[2], lo[2];
          relu_hi_lo(acc[j], hi, lo);
#pragma unroll
          for (int s = 0; s < 2; ++s) {
            a.out_hi[((blk0 + j) * 2 + s) * 64 + lane] = __builtin_bit_cast(bf16x8, hi[s]);
            a.out_lo[((blk0 + j) * 2 + s) * 64 + lane] = __builtin_bit_cast(bf16x8, lo[s]);
          }
        }
      }
    }
    cur = nxt;
  }
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // nothing may still be on its way into this workgroup's LDS
}

hipError_t launch_wide_mlp(const Plan &pl, const WideMlpLayer &l, hipStream_t st) {
  WideMlpArgs a;
  a.x = l.x;
  a.in_hi = static_cast<const bf16x8 *>(l.in_hi); a.in_lo = static_cast<const bf16x8 *>(l.in_lo);
  a.w1f = static_cast<const bf16x8 *>(l.w1f); a.wf = static_cast<const bf16x8 *>(l.wf);
  a.b1 = l.b1; a.bias = l.bias;
  a.h_hi = static_cast<bf16x8 *>(l.h_hi);
  a.out_hi = static_cast<bf16x8 *>(l.out_hi); a.out_lo = static_cast<bf16x8 *>(l.out_lo);
  a.out_u = static_cast<f32x4 *>(l.out_u); a.out_stat = l.out_stat;
  a.H = pl.H; a.K = l.K; a.NOUT = l.NOUT;
  a.n_tok = l.n_tok; a.n_tb = (l.n_tok + 31) / 32; a.R = l.R; a.G = pl.G;
  a.sb = pl.sb; a.sh = pl.sh; a.sn = pl.sn;
  a.n_tiles = (a.n_tb + 7) / 8;
  const int src = !l.x ? 2 : pl.f32 ? 1 : 0;
  // Blocks of eight output tiles, or of four, or both: a workgroup takes whole items, so the time goes in rounds of 256 of
  // them.  A round takes 20 units with blocks of eight, 13 with blocks of four (the first hidden layer and the barriers are not
  // halved), a second launch 4.  Where the width is an odd multiple of 128 the last block is one of four in any case, in a
  // launch of its own unless all are; otherwise the items beyond one or two whole rounds may be halved and go second (item i of
  // eight tiles is items 2 i and 2 i + 1 of four): 1 - 5 % of the forward with 2 .. 128 of them beyond one round, 1 - 3 % beyond
  // two, nothing or a loss of up to 4 % beyond four, where the workgroups that have one item less leave the others power.  Whole
  // forwards at rate 0, blocks of eight / four, us: 768-wide two-layer maps,
  // 40 tiles (120 items of eight) 193 / 168, 60 tiles (180) 208 / 236, 129 tiles (387) 336 / 398; 512-wide three-layer maps, 129
  // tiles (258) 371 / 358, 200 tiles (400) 412 / 484; 640-wide, 60 tiles (120 + 60) 243 / 207, 110 tiles (220 + 110) 276 / 290,
  // 140 tiles (280 + 140) 351 / 293.
  struct Launch { int nt, ob_first, n_ob, first, total; } launches[2];
  int n_launches = 0;
  {
    const int OB = a.NOUT / 32, tiles = a.n_tiles * pl.B * pl.H, i8 = tiles * (OB / 8), i4 = tiles * (OB / 4), rest = i8 % 256;
    const auto rounds = [](int items) { return (items + 255) / 256; };
    const int fours = rounds(i4) * 13, eights = rounds(i8) * 20 + (OB % 8 ? rounds(tiles) * 13 + 4 : 0);
    const bool halve = OB % 8 == 0 && i8 > 256 && i8 < 3 * 256 && rest > 0;
    const int both = halve ? i8 / 256 * 20 + rounds(2 * rest) * 13 + 4 : eights;
    if (OB < 8 || fours < (both < eights ? both : eights)) {
      launches[n_launches++] = {4, 0, OB / 4, 0, i4};
    } else if (both < eights) {
      launches[n_launches++] = {8, 0, OB / 8, 0, i8 - rest};
      launches[n_launches++] = {4, 0, OB / 4, 2 * (i8 - rest), 2 * rest};
    } else {
      launches[n_launches++] = {8, 0, OB / 8, 0, i8};
      if (OB % 8) launches[n_launches++] = {4, OB / 8 * 8, 1, 0, tiles};
    }
  }
  for (int i = 0; i < n_launches; ++i) {
    a.ob_first = launches[i].ob_first;
    a.n_ob = launches[i].n_ob;
    a.first = launches[i].first;
    a.total = launches[i].total;
    const int nwg = a.total < 256 ? (a.total + 7) / 8 * 8 : 256;               // one workgroup per CU
    // the longest ring that fits LDS and the shortest contraction of its instance
#define HA_WIDE_MLP(NT, SRC, NBUF) \
  do { \
    if (l.out_u && l.channel_lanes) wide_mlp_kernel<NT, SRC, 2, NBUF><<<nwg, 512, 0, st>>>(a); \
    else if (l.out_u) wide_mlp_kernel<NT, SRC, 1, NBUF><<<nwg, 512, 0, st>>>(a); \
    else wide_mlp_kernel<NT, SRC, 0, NBUF><<<nwg, 512, 0, st>>>(a); \
  } while (0)
#define HA_WIDE_MLP_SRC(NT, NBUF_X, NBUF_HBM) \
  do { \
    if (src == 0) HA_WIDE_MLP(NT, 0, NBUF_X); else if (src == 1) HA_WIDE_MLP(NT, 1, NBUF_X); else HA_WIDE_MLP(NT, 2, NBUF_HBM); \
  } while (0)
    if (a.K >= 256) { if (launches[i].nt == 8) HA_WIDE_MLP_SRC(8, 6, 9); else HA_WIDE_MLP_SRC(4, 9, 9); }
    else if (launches[i].nt == 8) HA_WIDE_MLP_SRC(8, 5, 5);
    else HA_WIDE_MLP_SRC(4, 5, 5);
#undef HA_WIDE_MLP_SRC
#undef HA_WIDE_MLP
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

}  // namespace ha
