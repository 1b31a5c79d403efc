// Query side of the hybrid-attention forward (Attention Surgery, Sec. 3.2, Eq. "hybrid"): the merging pass of split key ranges, which
// tiling of the query kernel a problem takes, and the instances with two waves per SIMD.  gfx950 only.
#include "ha_query_kernel.h"

namespace ha {

template <typename T>
static inline T *ws_ptr(void *ws, size_t off) { return reinterpret_cast<T *>(static_cast<char *>(ws) + off); }

// ------------------------------------------------------------------------------------------------
// merge_kernel: grid (n_tb, B*H), 4 waves, one 32-query block; wave w takes channels 32 w .. + 31.  The partial sums of the key
// ranges, put on their common maximum c_i, plus the precomputed linear part if there is one: y = (a + n) / (l + e).
// All ranges' loads are in flight at once: the pass is a few memory round trips long.
constexpr int kMaxSplit = 8;
template <bool F32>
__global__ __launch_bounds__(256) void merge_kernel(QueryArgs a) {
  constexpr int D = 128, RB = D / 32, ESZ = F32 ? 4 : 2, PITCH = 32 * ESZ + 16, CPR = 32 * ESZ / 16;
  __shared__ __align__(16) char stage_all[4 * 32 * PITCH];
  const int bh = blockIdx.y, tb = blockIdx.x, lane = threadIdx.x & 63, r = lane & 31, g = lane >> 5;
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int q0 = 32 * tb;
  const int64_t step = (int64_t)a.sp.BH * a.sp.n_tb, blk = (int64_t)bh * a.sp.n_tb + tb;
  const int n_split = a.sp.n_split;
  float ms[kMaxSplit], ls[kMaxSplit];
  f32x4 part[kMaxSplit][4], lin[4];
  float lin_e = 0.f;
#pragma unroll
  for (int s = 0; s < kMaxSplit; ++s) {
    const int64_t at = blk + (s < n_split ? s : 0) * step;          // (ranges there are not repeat the first, with weight 0)
    ms[s] = s < n_split ? a.sp.pm[at * 32 + r] : -INFINITY;
    ls[s] = a.sp.pl[at * 32 + r];
    if (s < n_split) {
      const f32x4 *src = reinterpret_cast<const f32x4 *>(a.sp.po) + (at * RB + w) * 4 * 64 + lane;
#pragma unroll
      for (int x4 = 0; x4 < 4; ++x4) part[s][x4] = src[x4 * 64];
    }
  }
#pragma unroll
  for (int x4 = 0; x4 < 4; ++x4) lin[x4] = f32x4{0.f, 0.f, 0.f, 0.f};
  if (a.lin) {
#pragma unroll
    for (int x4 = 0; x4 < 4; ++x4) lin[x4] = a.lin[((((int64_t)bh * a.n_tb + tb) * RB + w) * 4 + x4) * 64 + lane];
    lin_e = a.lin_e[(int64_t)bh * a.N + min(q0 + r, a.N - 1)];
  }
  float m = ms[0];
#pragma unroll
  for (int s = 1; s < kMaxSplit; ++s) m = fmaxf(m, ms[s]);
  float l = 0.f;
  f32x4 o[4] = {{0.f, 0.f, 0.f, 0.f}, {0.f, 0.f, 0.f, 0.f}, {0.f, 0.f, 0.f, 0.f}, {0.f, 0.f, 0.f, 0.f}};
#pragma unroll
  for (int s = 0; s < kMaxSplit; ++s)
    if (s < n_split) {
      const float wgt = fast_exp2((ms[s] - m) * a.sp.scale_log2e);
      l = __builtin_fmaf(wgt, ls[s], l);
#pragma unroll
      for (int x4 = 0; x4 < 4; ++x4)
#pragma unroll
        for (int j = 0; j < 4; ++j) o[x4][j] = __builtin_fmaf(wgt, part[s][x4][j], o[x4][j]);
    }
  const float den = l + lin_e, inv = 1.0f / den;
  if (w == 0) store_den(a, bh, lane, den, q0);
  char *stage = stage_all + w * 32 * PITCH;
#pragma unroll
  for (int x4 = 0; x4 < 4; ++x4) {
    const f32x4 y = {(o[x4][0] + lin[x4][0]) * inv, (o[x4][1] + lin[x4][1]) * inv, (o[x4][2] + lin[x4][2]) * inv, (o[x4][3] + lin[x4][3]) * inv};
    char *dst = stage + r * PITCH + (8 * x4 + 4 * g) * ESZ;
    if constexpr (F32) *reinterpret_cast<f32x4 *>(dst) = y;
    else *reinterpret_cast<bf16x4 *>(dst) = __builtin_convertvector(y, bf16x4);
  }
  asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");      // the wave's own staging area, in order (see store_tile)
  const int64_t base = (int64_t)(bh / a.H) * a.sb + (int64_t)(bh % a.H) * a.sh;
#pragma unroll
  for (int i = lane; i < 32 * CPR; i += 64) {
    const int row = i / CPR, ch = i % CPR;
    if (q0 + row < a.N) {
      const f32x4 piece = *reinterpret_cast<const f32x4 *>(stage + row * PITCH + ch * 16);
      char *dst = static_cast<char *>(a.out) + (base + (int64_t)(q0 + row) * a.sn + 32 * w) * ESZ + ch * 16;
      *reinterpret_cast<f32x4 *>(dst) = piece;
    }
  }
}

static QueryArgs query_args(const Plan &pl, const void *q, const ha_feature_map *phi_q, void *out, float *row_den, void *ws,
                            const WidePlan *wide) {
  const bool lin = wide || pl.split_linear;               // the linear part arrives precomputed
  QueryArgs a;
  a.q = q;
  a.out = out;
  a.row_den = row_den;
  a.lin = wide ? ws_ptr<f32x4>(ws, wide->off_lin) : lin ? ws_ptr<f32x4>(ws, pl.off_lin) : nullptr;
  a.lin_e = wide ? ws_ptr<float>(ws, wide->off_e) : lin ? ws_ptr<float>(ws, pl.off_e) : nullptr;
  a.n_tb = wide ? wide->n_tb_q : pl.n_tb;
  a.ks_frag = ws_ptr<bf16x8>(ws, pl.off_ks);
  a.vs_frag = ws_ptr<bf16x8>(ws, pl.off_vs);
  a.w1f = ws_ptr<bf16x8>(ws, pl.off_w1q);
  a.w2f = ws_ptr<bf16x8>(ws, pl.off_w2q);
  a.b1 = phi_q ? phi_q->b1 : nullptr;
  a.b2 = phi_q ? phi_q->b2 : nullptr;
  a.st_hi = ws_ptr<bf16x8>(ws, pl.off_sthi);
  a.st_lo = ws_ptr<bf16x8>(ws, pl.off_stlo);
  a.z = ws_ptr<float>(ws, pl.off_z);
  a.H = pl.H; a.N = pl.N; a.NS = pl.NS;
  a.CC = pl.CC; a.n_cc = pl.n_cc; a.R = pl.R; a.G = pl.G; a.LW = pl.LW;
  a.n_ktiles = pl.n_ktiles; a.n_kblocks = pl.n_kblocks;
  a.has_linear = pl.NL > 0; a.P = pl.P; a.act = pl.act_q;
  a.sb = pl.sb; a.sh = pl.sh; a.sn = pl.sn;
  a.scale_log2e = pl.scale * kLog2e;
  a.sp = SplitArgs{nullptr, nullptr, nullptr, 1, 0, 0, 0.f};
  return a;
}

enum class Tiling { kAlone, kSmall, kLarge };
static Tiling tiling_of(const Plan &pl, bool lin) {
  // Three tilings of one computation (every query column sees the same keys in the same order): 4 waves x 32 queries, one wave per
  // SIMD, with a ring of 8 key blocks (ha_query_alone.hip); 8 waves x 32 queries with that ring and a barrier every 64 keys, one
  // workgroup per CU; and 4 waves x 32 queries with a ring of 4 and a barrier every 32 keys, two workgroups per CU.  The variants'
  // tiles are part of their definition, so block_size decides there between the latter two; for the plain operator the sizes do.
  //   128-query tiles that do not outnumber the CUs: a workgroup has a CU to itself, so that one wave per SIMD for the keys, with the map
  // in waves of its own, is best.  Whole calls, us, better one of the other two / alone: H = 12, R = 4, d = 128: N = 300 (B = 2)
  // 35.3 / 30.0, 1560  43.1 / 33.9, 2600  48.5 / 39.9; H = 8, N = 3900, R = 2  69.8 / 57.4; two workgroups more than CUs (H = 6,
  // N = 5400, R = 3)  69.0 / 86.3; d = 64: H = 2, N = 1024, fp32  22.8 / 18.5, H = 12, N = 2600, R = 2  40.0 / 32.2; rate 1: H = 8,
  // N = 4000  76.9 / 72.6, d = 64, H = 4, N = 4000  56.4 / 47.2.  With the linear part precomputed a short loop is as long either way
  // (6 key blocks 72.4 / 73.2, 13 68.5 / 68.5), a long one shorter (94: 106.1 / 104.1).
  const auto wgs = [&](int qt) { return (int64_t)((pl.N + qt - 1) / qt) * pl.B * pl.H; };
  const int64_t nblk = (pl.NS + 31) / 32;
  const bool alone = pl.CC == 0 && pl.LW == 0 && wgs(128) <= 256 && (!lin || nblk >= 20);
  //   Otherwise, d = 128, maps in the epilogue: the 4-wave kernel reads their operands from L2 instead of LDS and fetches every key
  // block twice as often, so it is better only where its last round of workgroups is emptier.  In us: a round of 256 large
  // workgroups takes 0.50 per key block and 14 beside, one of 512 small ones 0.52 and 24, a last one of at most 256 small ones
  // 0.30 and 26 (877 problems timed with both, R = 2 .. 16, both dtypes: 63 of them take the small tiles; none is more than
  // 0.4 % slower than with large ones throughout, none more than 2.3 % than with small ones).  Whole calls, large / small:
  // H = 10, N = 6500, R = 2 (260 / 510 workgroups) 196 / 149; H = 20, N = 3200, R = 4 (260 / 500) 94 / 81; H = 12, N = 5504, R = 2
  // (264 / 516) 175 / 175; H = 64, N = 5556, R = 2 (1408 / 2816) 577 / 614.  Within one round of large ones those are better.
  //   d = 128, linear part precomputed or absent: no operands to fetch.  In hundredths of a key block a round of large workgroups
  // takes 100 per block, one of small ones 105, a last one of at most 256 small ones 65; a short loop's start costs the large
  // ones 65 more, and 250 with every further round (small workgroups start where one has ended).  (660 problems timed with both:
  // the choice is on average 0.1 % off the better one, at most 4.6 %.)  Large / small, R = 1: H = 250, N = 457 (500 / 1000)
  // 71.7 / 63.6; H = 128, N = 268 (256 / 384) 35.2 / 33.3; H = 86, N = 3975, fp32 (1376 / 2752) 725 / 759; 256-wide maps: H = 48,
  // N = 4818, R = 16 (912 / 1824) 342 / 323.
  //   d = 64: everything is small, and two independent workgroups per CU fill each other's gaps once there is more than one round
  // of large ones (R = 2 .. 16: large takes 0.85 - 0.97 of small's time within one round of them, 0.96 - 1.24, on average 1.06, beyond).
  const int64_t rounds = (wgs(256) + 255) / 256, full = wgs(128) / 512, tail = wgs(128) % 512;
  bool big;
  if (alone) big = false;
  else if (pl.LW > 0 || pl.CC > 0) big = pl.KT == 128;
  else if (pl.D == 64) big = wgs(256) <= 256;
  else if (lin || pl.NL == 0) {
    const int64_t len = nblk > 0 ? nblk : 1024;              // (rate 0: the rounds alone count)
    big = rounds * (100 * len + 250) - 185 <= full * 105 * len + (tail == 0 ? 0 : tail <= 256 ? 65 : 105) * len;
  } else {
    const int64_t last = tail == 0 ? 0 : tail <= 256 ? 30 * nblk + 2600 : 52 * nblk + 2400;
    big = wgs(256) <= 256 || rounds * (50 * nblk + 1400) <= full * (52 * nblk + 2400) + last;
  }
  return alone ? Tiling::kAlone : big ? Tiling::kLarge : Tiling::kSmall;
}

hipError_t launch_query(const Plan &pl, const void *q, const ha_feature_map *phi_q, void *out, float *row_den, void *ws,
                        hipStream_t st, const WidePlan *wide) {
  if (!wide && query_side_is_linear(pl)) return launch_linear_query(pl, q, *phi_q, out, row_den, ws, st);
  const bool lin = wide || pl.split_linear;
  QueryArgs a = query_args(pl, q, phi_q, out, row_den, ws, wide);
  if (pl.n_split > 1) {
    // (choose_split says when)
    a.sp = split_args(pl, ws);
    a.n_qtiles = (pl.N + 255) / 256;
    a.total_wg = a.n_qtiles * pl.B * pl.H * pl.n_split;
    const dim3 grid((a.total_wg + 7) / 8 * 8), mgrid((pl.N + 31) / 32, pl.B * pl.H);
    if (pl.f32) query_kernel_ring<128, 128, 128, 8, 8, 2, true, true, 3><<<grid, 512, 0, st>>>(a);
    else query_kernel_ring<128, 128, 128, 8, 8, 2, false, true, 3><<<grid, 512, 0, st>>>(a);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    if (pl.f32) merge_kernel<true><<<mgrid, 256, 0, st>>>(a);
    else merge_kernel<false><<<mgrid, 256, 0, st>>>(a);
    return hipGetLastError();
  }
  const Tiling tiling = tiling_of(pl, lin);
  const bool big = tiling == Tiling::kLarge;
  const int qt = big ? 256 : 128;
  a.n_qtiles = (pl.N + qt - 1) / qt;
  a.total_wg = a.n_qtiles * pl.B * pl.H;
  dim3 grid(((a.total_wg + 7) / 8) * 8);
  if (tiling == Tiling::kAlone) return launch_query_alone(pl, a, grid, st);
#define HA_QUERY(DD, HH, FF, F32) \
  do { \
    if (pl.LW > 0) { \
      if (big) query_kernel_ring<DD, HH, FF, 8, 8, 2, F32, false, 2><<<grid, 512, 0, st>>>(a); \
      else query_kernel_ring<DD, HH, FF, 4, 4, 1, F32, false, 2><<<grid, 256, 0, st>>>(a); \
    } else if (pl.CC > 0) { \
      if (big) query_kernel_ring<DD, HH, FF, 8, 8, 2, F32, false, 1><<<grid, 512, 0, st>>>(a); \
      else query_kernel_ring<DD, HH, FF, 4, 4, 1, F32, false, 1><<<grid, 256, 0, st>>>(a); \
    } else if constexpr (HH <= 128) { \
      if (big) query_kernel_ring<DD, HH, FF, 8, 8, 2, F32><<<grid, 512, 0, st>>>(a); \
      else query_kernel_ring<DD, HH, FF, 4, 4, 1, F32><<<grid, 256, 0, st>>>(a); \
    } else { \
      return hipErrorInvalidValue;      /* the plan of the plain operator has the wider maps' linear part precomputed */ \
    } \
  } while (0)
  if (lin) {
    if (big) {
      if (pl.f32) query_kernel_ring<128, 128, 128, 8, 8, 2, true, true><<<grid, 512, 0, st>>>(a);
      else query_kernel_ring<128, 128, 128, 8, 8, 2, false, true><<<grid, 512, 0, st>>>(a);
    } else {
      if (pl.f32) query_kernel_ring<128, 128, 128, 4, 4, 1, true, true><<<grid, 256, 0, st>>>(a);
      else query_kernel_ring<128, 128, 128, 4, 4, 1, false, true><<<grid, 256, 0, st>>>(a);
    }
  }
  else if (pl.D == 64) { if (pl.f32) HA_QUERY(64, 64, 64, true); else HA_QUERY(64, 64, 64, false); }
  else if (pl.HD == 128) { if (pl.f32) HA_QUERY(128, 128, 128, true); else HA_QUERY(128, 128, 128, false); }
  else { if (pl.f32) HA_QUERY(128, 256, 256, true); else HA_QUERY(128, 256, 256, false); }
#undef HA_QUERY
  return hipGetLastError();
}

// Two forwards of one problem, the softmax teacher's and the student's, as one launch: the student's workgroups start on the CUs that the
// teacher's last round leaves idle.
// Estimated, in us, for n workgroups each: a key block 0.50 (d = 64: 0.30), 0.42 (0.25) in a round of up to 150 workgroups, more towards
// 256; beside the loop 5 (4) for the teacher, 14 (7) for the student, whose epilogue evaluates the map.  One after the other: whole
// rounds.  In one launch: every CU takes the next workgroup when it is free.  The estimate has to be 4 % better, and the keys of the
// heads that an XCD works on must not outgrow its 4 MiB of L2 by the student's share alone (H = 12, N = 3500: 155.7 / 163.1 at R = 3).
// Whole losses, one after the other / in one launch, us: H = 12, N = 2900, R = 8 122 / 107; H = 12, N = 9361, R = 8 610 / 597; H = 8, N = 5000, R = 3
// 189 / 164; H = 5, N = 7000, R = 5 214 / 188; d = 64, H = 12, N = 4000, R = 5 108.5 / 94.6; not taken: H = 5, N = 9361, R = 2 353 / 378; H = 8, N = 15000,
// R = 5 976 / 997; H = 12, N = 5000, R = 5 (240 workgroups) 218.6 / 215.4.  (81 sizes; the estimate was off by 10 us where it did not hold.)
static int64_t large_tiles(const Plan &pl) { return (int64_t)((pl.N + 255) / 256) * pl.B * pl.H; }
bool query_pair_fits(const Plan &teacher, const Plan &student) {
  const bool square = student.HD == student.D && student.F == student.D && student.DM == 0;
  if (student.NL == 0 || student.NS == 0 || !square || student.split_linear || student.CC > 0 || student.LW > 0) return false;
  // (beyond four rounds a last one that is not full is little, and the teacher's keys would be held beside the student's for it)
  if (teacher.n_split > 1 || student.n_split > 1 || large_tiles(teacher) > 1024 || tiling_of(teacher, false) != Tiling::kLarge ||
      tiling_of(student, false) != Tiling::kLarge)
    return false;
  const int n = (int)large_tiles(teacher), whole = n / 256, rest = n % 256;
  const bool d64 = teacher.D == 64;
  const double full = d64 ? 0.30 : 0.50, light = d64 ? 0.25 : 0.42;
  const double last = light + (full - light) * (rest > 150 ? (rest - 150) / 106.0 : 0.0);
  const int blocks[2] = {(teacher.NS + 31) / 32, (student.NS + 31) / 32};
  const double beside[2] = {d64 ? 4.0 : 5.0, d64 ? 7.0 : 14.0};
  double apart = 2.0, one[2];                             // (a launch more)
  for (int i = 0; i < 2; ++i) {
    one[i] = full * blocks[i] + beside[i];
    apart += whole * one[i] + (rest ? last * blocks[i] + beside[i] : 0.0);
  }
  // together: 256 - rest CUs are free for the student after `whole` rounds of the teacher, the others a round later
  const double at[2] = {whole * one[0], (whole + (rest ? 1 : 0)) * one[0]};
  auto done = [&](double t) {                             // workgroups of the student that have ended by then
    int64_t c = 0;
    for (int i = 0; i < 2; ++i)
      if (t >= at[i]) c += (i ? rest : 256 - rest) * (int64_t)((t - at[i]) / one[1] + 1e-6);
    return c;
  };
  double together = 1e30;
  for (double start : at) {
    double t = start;
    while (done(t) < n) t += one[1];
    together = t < together ? t : together;
  }
  if (together < at[1]) together = at[1];
  const int64_t per_head = (teacher.N + 255) / 256, heads = ((n + 7) / 8 + per_head - 1) / per_head, l2 = 4 << 20;
  const int64_t keys = heads * teacher.N * (4 * teacher.D);   // K and V of those heads in bf16
  if (keys <= l2 && keys + heads * student.NS * (4 * student.D) > l2) return false;
  return together <= 0.96 * apart;
}
hipError_t launch_query_pair(const Plan &teacher, const Plan &student, const void *q, const ha_feature_map &phi_q, void *y_teacher,
                             void *y_student, float *row_den, void *ws_teacher, void *ws_student, hipStream_t st) {
  QueryPair p;
  p.a[0] = query_args(teacher, q, nullptr, y_teacher, nullptr, ws_teacher, nullptr);
  p.a[1] = query_args(student, q, &phi_q, y_student, row_den, ws_student, nullptr);
  for (QueryArgs &a : p.a) {
    a.n_qtiles = (teacher.N + 255) / 256;
    a.total_wg = (int)large_tiles(teacher);
  }
  p.n_first = (p.a[0].total_wg + 7) / 8 * 8;
  const dim3 grid(2 * p.n_first);
  if (teacher.D == 64) {
    if (teacher.f32) query_pair_kernel<64, true><<<grid, 512, 0, st>>>(p);
    else query_pair_kernel<64, false><<<grid, 512, 0, st>>>(p);
  } else {
    if (teacher.f32) query_pair_kernel<128, true><<<grid, 512, 0, st>>>(p);
    else query_pair_kernel<128, false><<<grid, 512, 0, st>>>(p);
  }
  return hipGetLastError();
}

}  // namespace ha
