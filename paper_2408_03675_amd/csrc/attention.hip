// Causal attention of the prefill with each query row's log-sum-exp: the
// forward pass of FlashAttention-2 that Appendix A.7 reuses, whose
// log-sum-exp lets the proxy-token score run as the single column reduction
// of Algorithm 2 (nacl_score's lse argument).  bf16 Q, K, V and output,
// fp32 accumulation, head dim 64 or 128, grouped query heads.
//
// A work-group's waves each take 64 consecutive query rows of one query head
// (two 32-row MFMA tiles, Q in registers) and stream the head's keys in tiles
// of 64 together:
//   S^T = K Q^T      v_mfma_f32_32x32x16_bf16, keys as MFMA rows, so lane
//                    (hl, r) holds keys 8 i + 4 hl .. + 3 of each 32-key block
//                    for query r: a lane owns one query per tile, and the
//                    reference, the sum and the rescale are per-lane scalars
//                    (the two lane halves agree through one permlane swap)
//   O^T += V^T P^T   the exponentials P in bf16 as the B operand straight
//                    from the S^T registers, V^T by transposing LDS reads of
//                    the same keys (a permutation of the contraction).
//
// What bounds it, and why it looks like this.  Per 64-key tile a wave has 64
// MFMAs (32 cycles each) and, for each of a lane's 64 logits, an FMA, an
// exponential, an addition and half a maximum and conversion.
// - 64 rows per wave: an LDS fragment then serves two MFMAs of 32 cycles, 64
//   bytes per cycle and CU where 32 rows take 128, all the LDS delivers (the
//   kernel with 32 rows per wave waited for LDS: 2350 of 4700 cycles per
//   64-row tile without an instruction).  It takes 64 + 128 accumulation
//   registers for Q and O and about 250 vector registers for two tiles of
//   logits: one wave per SIMD.
// - With one wave per SIMD, matrix and vector work overlap only within the
//   wave: a software pipeline runs the logits of tile j + 1 beside the
//   exponentials of tile j, and the value products of tile j beside its row
//   sums and the maxima of tile j + 1.  AttnPlan deals the vector operations
//   to half steps of one MFMA each, equal in issue cycles, and
//   sched_barriers keep them there.  3180 cycles per tile of which the matrix
//   unit is busy for 2050 (32k rows, D = 128).
// - The running maximum is only a reference: it stays until a logit exceeds
//   it by 2^8 (the sums and P scale with it exactly), so the output is
//   rescaled in a rare branch and not in the loop.
// - K and V go from memory to LDS by DMA (buffer loads with the lds flag),
//   two tiles of each, spread over the half steps; the loop has one barrier
//   per tile, in the middle: K is loaded two tiles ahead of its use and V
//   one, K's last fragments are in registers when the barrier is passed.
// 32k rows, 128 heads of 128: 35.4 ms before (16x16x32 MFMAs, 32 rows per
// wave, 0.99 PFLOP/s), 27.7 ms now (1.27 PFLOP/s; a plain bf16 product of
// 16384^3 reaches 1.36 on this part: the clock falls from 2.16 to 1.8 GHz
// under the denser matrix work).

#include <type_traits>

#include "device_common.h"
#include "internal.h"

namespace nacl {

namespace {

constexpr int kAttnKeys = 64;   // keys per tile
constexpr int kRsrcWord3 = 0x00020000;

typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
// Calls f(std::integral_constant<int, i>) for i = I .. N-1.
template <int N, int I = 0, class F>
__device__ __forceinline__ void static_for(F&& f) {
  if constexpr (I < N) {
    f(std::integral_constant<int, I>{});
    static_for<N, I + 1>(f);
  }
}

// One buffer load that writes 1 KB of LDS (16 bytes per lane, lane order)
// at byte lds of the work-group's allocation.  An asm block, so that the
// compiler does not make LDS reads of the tile in hand wait for the loads of
// the next one; the kernel waits for them itself (wait_dma).
__device__ __forceinline__ void dma_1k(u32x4 rsrc, uint32_t voff, uint32_t off, uint32_t lds) {
  uint32_t t;
  asm volatile("s_mov_b32 m0, %1\n\tv_add_u32 %0, %2, %3\n\tbuffer_load_dwordx4 %0, %4, 0 offen lds"
               : "=&v"(t)
               : "s"(lds), "s"(off), "v"(voff), "s"(rsrc)
               : "memory");
}
// Every DMA of this wave and every LDS read it issued has completed, then
// the work-group's barrier.
__device__ __forceinline__ void dma_barrier() {
  asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier" ::: "memory");
}

typedef float f32x16 __attribute__((ext_vector_type(16)));

// acc += A B on the accumulation registers, where the output stays so that the
// vector registers hold two tiles of logits.  The compiler does not know an
// asm block's wait states: anything else that touches an accumulator goes
// through settle() first, and an operand written by a vector instruction is
// written at least two instructions before (a tile's probabilities: at least
// one half step).
__device__ __forceinline__ void mfma_acc(f32x16& acc, bf16x8 fa, u32x4 fb) {
  asm volatile("v_mfma_f32_32x32x16_bf16 %0, %1, %2, %0" : "+a"(acc) : "v"(fa), "v"(fb));
}
// Every MFMA issued before has written its accumulator (32 wait states; a
// 32x32x16 needs 18), and the accumulators are in accumulation registers.
__device__ __forceinline__ void settle(f32x16 (&acc)[2][2]) {
  asm volatile("s_nop 15\n\ts_nop 15" : "+a"(acc[0][0]), "+a"(acc[0][1]), "+a"(acc[1][0]), "+a"(acc[1][1]));
}
__device__ __forceinline__ void settle(f32x16 (&acc)[4][2]) {
  asm volatile("s_nop 15\n\ts_nop 15"
               : "+a"(acc[0][0]), "+a"(acc[0][1]), "+a"(acc[1][0]), "+a"(acc[1][1]), "+a"(acc[2][0]), "+a"(acc[2][1]),
                 "+a"(acc[3][0]), "+a"(acc[3][1]));
}

// Where a tile's vector work stands: first operation of each kind at half step
// t (one MFMA each; HA beside S^T, then HB beside O^T).  A wave issues one
// instruction in about 4.75 cycles (9.5 for an exponential) and the matrix
// unit takes 32 per MFMA, so each half step is filled up to the same share.
template <int HA, int HB, int kReadsA, int kReadsB, int kDmaN>
struct AttnPlan {
  int f[HA + HB + 1] = {}, e[HA + HB + 1] = {}, c[HA + HB + 1] = {}, x[HA + HB + 1] = {}, s[HA + HB + 1] = {};
  // LDS reads of the next group of fragments: in the first half steps of a group.
  static constexpr int reads(int t) {
    const int ga = HA / 4, gb = HB / 4;
    if (t < HA) {
      const bool k = t / ga < 3;  // the last group of S^T reads the first of V
      return t % ga < (k ? kReadsA : kReadsB) ? (k ? 1 : 2) : 0;
    }
    const bool v = (t - HA) / gb < 3;
    return (t - HA) % gb < (v ? kReadsB : kReadsA) ? (v ? 2 : 1) : 0;
  }
  // DMA loads: every second half step from the barrier on (every one if there are few).
  static constexpr int dma(int t) {
    const int t0 = HA - HA / 4, d = t - t0;
    const int stride = kDmaN * 2 <= HA / 4 + HB ? 2 : 1;
    return d >= 0 && d % stride == stride - 1 && d / stride < kDmaN ? d / stride : -1;
  }
  static constexpr int kX0 = HA + 4;  // the next tile's logits are complete
  constexpr AttnPlan() {
    constexpr int one = 19, ex = 32, T = HA + HB;  // quarter cycles
    int total = 64 * (one + ex + one) + 32 * 2 * one + 8 * one;
    for (int t = 0; t < T; ++t) total += reads(t) * one + (dma(t) >= 0 ? 3 * one : 0);
    const int cap = (total + T - 1) / T + 2;
    int nf = 0, ne = 0, nc = 0, nx = 0, ns = 0;
    for (int t = 0; t < T; ++t) {
      f[t] = nf, e[t] = ne, c[t] = nc, x[t] = nx, s[t] = ns;
      int left = cap - reads(t) * one - (dma(t) >= 0 ? 3 * one : 0);
      const int e2 = t >= 2 ? e[t - 1] : 0, f1 = f[t];  // exponentials two half steps old, FMAs one
      bool more = true;
      while (more) {
        more = false;
        if (nc < 32 && 2 * nc + 2 <= e2 && left >= one) ++nc, left -= one, more = true;
        if (ne < 64 && ne < f1 && left >= ex) ++ne, left -= ex, more = true;
        if (nf < 64 && nf < ne + 4 && left >= one) ++nf, left -= one, more = true;
      }
      while (t >= kX0 && nx < 32 && left >= one) ++nx, left -= one;
      while (ns < 64 && ns < e2 && left >= one && (ne == 64 || t >= HA - HA / 4)) ++ns, left -= one;
    }
    f[T] = 64, e[T] = 64, c[T] = 32, x[T] = 32, s[T] = 64;  // what is left: the last half step
  }
};

// NW waves of 64 query rows per work-group.
template <int D, int NW>
__global__ __launch_bounds__(64 * NW, 1) void attn_fwd_kernel(AttnLaunch a) {
  constexpr int kRowBytes = D * 2;         // one K or V row
  constexpr int kChunks = kRowBytes / 16;  // 16-byte chunks per row
  constexpr int kSwz = kChunks - 1;
  constexpr int kTile = kAttnKeys * kRowBytes;
  constexpr int kC = D / 16;               // contraction steps of S^T
  constexpr int kDt = D / 32;              // 32-wide d tiles of O^T
  constexpr int kDma = kTile / 1024 / NW;  // 1 KB loads per wave and tile
  constexpr int kRows = 64 * NW;           // query rows per work-group
  constexpr int kRpi = 1024 / kRowBytes;   // rows per 1 KB load
  constexpr int kSA = 2 * kC, kSB = 4 * kDt;  // fragment steps of S^T and of O^T (two MFMAs each)
  constexpr int kGA = kSA / 4, kGB = kSB / 4;  // fragments per group (four groups of each)
  // K tiles of both parities, then V tiles of both parities.
  __shared__ __attribute__((aligned(1024))) unsigned char smem[4 * kTile];
  const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) unsigned char*)smem;

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int hl = lane >> 5, m32 = lane & 31;

  // Work-groups are dealt to the 8 XCDs in turn: XCD x takes its share of
  // the tiles of the heads that 8 does not divide, then heads x * heads_x ..
  // in groups of `group` heads (whose K and V share its L2), the longest
  // tiles of a group first.
  const int xcd = blockIdx.x & 7, n_heads = a.B * a.H * a.G, rest0 = 8 * a.heads_x, n_rest = n_heads - rest0;
  const int rest = (n_rest * a.n_tiles - xcd + 7) / 8;  // of the remaining heads' tiles
  int slot = blockIdx.x >> 3, bhq, tile;
  if (slot < rest) {
    const int u = 8 * slot + xcd;
    tile = a.n_tiles - 1 - u / n_rest;
    bhq = rest0 + u % n_rest;
  } else {
    slot -= rest;
    if (slot >= a.heads_x * a.n_tiles) return;
    const int g0 = slot / (a.group * a.n_tiles) * a.group, gn = min(a.group, a.heads_x - g0);
    const int i = slot - g0 * a.n_tiles;
    tile = a.n_tiles - 1 - i / gn;
    bhq = xcd * a.heads_x + g0 + i % gn;
  }
  const int Hq = a.H * a.G;
  const int b = bhq / Hq, hq = bhq - b * Hq, h = hq / a.G;
  const int L = a.L;
  const int q0 = tile * kRows;
  const int qw0 = q0 + 64 * wave;
  const int n_kv = (min(q0 + kRows, L) + kAttnKeys - 1) / kAttnKeys;
  // Tiles this wave's rows see: the last one holds its diagonal.
  const int n_w = qw0 < L ? qw0 / kAttnKeys + 1 : 0;

  const __bf16* qh = a.q + (int64_t)b * a.qs[0] + (int64_t)hq * a.qs[1];
  const __bf16* kh = a.k + (int64_t)b * a.ks[0] + (int64_t)h * a.ks[1];
  const __bf16* vh = a.v + (int64_t)b * a.vs[0] + (int64_t)h * a.vs[1];
  const uint32_t qrow = (uint32_t)a.qs[2] * 2u, krow = (uint32_t)a.ks[2] * 2u, vrow = (uint32_t)a.vs[2] * 2u;
  // Rows at or past L read as zeros through the descriptors' ranges.
  const __amdgpu_buffer_rsrc_t qr = __builtin_amdgcn_make_buffer_rsrc(const_cast<__bf16*>(qh), (short)0,
                                                                      (int)((uint32_t)L * qrow), kRsrcWord3);
  auto words = [](const __bf16* base, uint32_t bytes) {
    const uint64_t p = (uint64_t)base;
    return u32x4{(uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)p),
                 (uint32_t)__builtin_amdgcn_readfirstlane((int)((uint32_t)(p >> 32) & 0xFFFFu)),
                 (uint32_t)__builtin_amdgcn_readfirstlane((int)bytes), (uint32_t)kRsrcWord3};
  };
  const u32x4 kr = words(kh, (uint32_t)L * krow), vr = words(vh, (uint32_t)L * vrow);

  // DMA: load i of this wave's share fills kRpi rows of the
  // tile; the 16 bytes at chunk position x of row r are the row's chunk
  // x ^ (r & kSwz) for K (the rows of a fragment read fall on distinct
  // banks) and x ^ ((r & 3) << 1) for V (the four rows of a transposed read).
  uint32_t kvo[kDma], vvo[kDma];
#pragma unroll
  for (int i = 0; i < kDma; ++i) {
    const int r = (wave * kDma + i) * kRpi + lane / kChunks, x = lane % kChunks;
    kvo[i] = (uint32_t)r * krow + (uint32_t)((x ^ (r & kSwz)) * 16);
    vvo[i] = (uint32_t)r * vrow + (uint32_t)((x ^ ((r & 3) << 1)) * 16);
  }
  // Load i of tile j's K or V into the buffer of its parity (none past the last tile).
  auto dma_k = [&](int j, int i) {
    dma_1k(kr, kvo[i], j < n_kv ? (uint32_t)(j * kAttnKeys) * krow : 0x80000000u,
           lds0 + (j & 1) * kTile + (wave * kDma + i) * 1024);
  };
  auto dma_v = [&](int j, int i) {
    dma_1k(vr, vvo[i], j < n_kv ? (uint32_t)(j * kAttnKeys) * vrow : 0x80000000u,
           lds0 + (2 + (j & 1)) * kTile + (wave * kDma + i) * 1024);
  };
#pragma unroll
  for (int i = 0; i < kDma; ++i) dma_k(0, i);
#pragma unroll
  for (int i = 0; i < kDma; ++i) dma_k(1, i);

  // Q fragments (B operand of S^T): query row qw0 + 32 qt + m32, d = 16 c + 8 hl .. + 7.
  bf16x8 qf[2][kC];
#pragma unroll
  for (int qt = 0; qt < 2; ++qt) {
    const int row = qw0 + 32 * qt + m32;
    const uint32_t ro = row < L ? (uint32_t)row * qrow : 0x80000000u;  // past the range: zeros
#pragma unroll
    for (int c = 0; c < kC; ++c)
      qf[qt][c] = __builtin_bit_cast(bf16x8, __builtin_amdgcn_raw_buffer_load_b128(qr, ro + (uint32_t)(32 * c + 16 * hl), 0, 0));
  }

  // Kept in accumulation registers (an MFMA operand reads them there): the
  // vector registers are for the logits.
#pragma unroll
  for (int qt = 0; qt < 2; ++qt)
#pragma unroll
    for (int c = 0; c < kC; ++c) asm volatile("" : "+a"(qf[qt][c]));

  // Fragment addresses.  K (A operand of S^T): row 32 kt + m32, chunk
  // 2 c + hl.  V^T (A operand of O^T): the 16 lanes of a group read 4 keys x
  // 16 d and receive the transpose, d = 32 dt + m32 and keys 16 ks + 8 jh +
  // 4 hl .. + 3: the keys that lane half hl's logits hold.
  uint32_t ka[kC], va[kDt];
#pragma unroll
  for (int c = 0; c < kC; ++c) ka[c] = (uint32_t)(m32 * kRowBytes + (((2 * c + hl) ^ (m32 & kSwz)) * 16));
  {
    const int i = lane & 15, mh = (lane >> 4) & 1, key = 4 * hl + (i >> 2);
#pragma unroll
    for (int dt = 0; dt < kDt; ++dt)
      va[dt] = (uint32_t)(key * kRowBytes + (((4 * dt + 2 * mh + ((i & 3) >> 1)) ^ ((key & 3) << 1)) * 16) + (i & 1) * 8);
  }
  auto kfrag = [&](auto par_c, auto f_c) {  // fragment f: c = f / 2, kt = f % 2
    constexpr int f = decltype(f_c)::value;
    return __builtin_bit_cast(bf16x8, *reinterpret_cast<const u32x4*>(smem + ka[f / 2] + decltype(par_c)::value * kTile +
                                                                      (f % 2) * 32 * kRowBytes));
  };
  auto vfrag = [&](auto par_c, auto f_c) {  // fragment f: ks = f / kDt, dt = f % kDt
    constexpr int f = decltype(f_c)::value;
    typedef short s16x4 __attribute__((ext_vector_type(4)));
    const unsigned char* p = smem + va[f % kDt] + (2 + decltype(par_c)::value) * kTile + (f / kDt) * 16 * kRowBytes;
    union { s16x4 h[2]; bf16x8 v; } u;
    u.h[0] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4*)p);
    u.h[1] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4*)(p + 8 * kRowBytes));
    return u.v;
  };

  const float c2 = a.c2;
  f32x16 acc[kDt][2];  // O^T
#pragma unroll
  for (int dt = 0; dt < kDt; ++dt)
#pragma unroll
    for (int qt = 0; qt < 2; ++qt)
#pragma unroll
      for (int i = 0; i < 16; ++i) acc[dt][qt][i] = 0.f;
  settle(acc);
  float m[2] = {0.f, 0.f}, l[2] = {0.f, 0.f};
  f32x16 s0[2][2], s1[2][2];  // S^T tiles [kt][qt] of the tile in hand and the next
  bf16x8 fr[2][4];  // fragment groups: the one in use and the next

  // Key 32 kt + 8 (i / 4) + 4 hl + i % 4 of the diagonal tile is past row
  // 32 qt + m32 (both from the wave's first row).
  auto mask = [&](f32x16 (&s)[2][2]) {
#pragma unroll
    for (int kt = 0; kt < 2; ++kt)
#pragma unroll
      for (int qt = 0; qt < 2; ++qt) {
        const int lim = 32 * qt + m32 - 32 * kt - 4 * hl;
#pragma unroll
        for (int i = 0; i < 16; ++i)
          if (8 * (i / 4) + i % 4 > lim) s[kt][qt][i] = -INFINITY;
      }
  };
  auto half_max = [&](float x) {
    auto p = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    return fmaxf(__uint_as_float(p[0]), __uint_as_float(p[1]));
  };

  // The middle of tile j: every wave has read K of tile j + 1 and V of tile
  // j - 1, and the loads issued one tile earlier (K of j + 2, V of j) have landed.
  auto middle = [&](int j) {
    dma_barrier();
#pragma unroll
    for (int i = 0; i < kDma; ++i) dma_k(j + 3, i);
#pragma unroll
    for (int i = 0; i < kDma; ++i) dma_v(j + 1, i);
  };

  // One tile: the exponentials of s (tile j) beside the logits of tile j + 1
  // (into sn), then the value products of tile j beside the row sums and the
  // maximum of sn.  Every half step is one MFMA and its share of the vector
  // work, fenced so that the compiler keeps them side by side.
  auto step = [&](auto par_c, f32x16 (&s)[2][2], f32x16 (&sn)[2][2], int j) {
    constexpr int PAR = decltype(par_c)::value;
    using KP = std::integral_constant<int, 1 - PAR>;
    using VP = std::integral_constant<int, PAR>;
    u32x4 pf[4][2];  // P^T fragments [ks][qt]
    // Logits in the order the value products need them: group v / 8 is
    // (ks, qt), element v % 8 of it.  The exponent's FMA, the exponential and
    // the conversion of a logit stand a half step apart, so that none waits
    // for the one before it.
    auto vfma = [&](auto v_c) {
      constexpr int v = decltype(v_c)::value, ks = v / 16, qt = (v / 8) % 2, i = 8 * (ks % 2) + v % 8;
      float x = __builtin_fmaf(s[ks / 2][qt][i], c2, -m[qt]);
      asm volatile("" : "+v"(x));
      s[ks / 2][qt][i] = x;
    };
    auto vexp = [&](auto v_c) {
      constexpr int v = decltype(v_c)::value, ks = v / 16, qt = (v / 8) % 2, i = 8 * (ks % 2) + v % 8;
      float x = __builtin_amdgcn_exp2f(s[ks / 2][qt][i]);
      asm volatile("" : "+v"(x));
      s[ks / 2][qt][i] = x;
    };
    auto vcvt = [&](auto p_c) {  // the pair of logits 2 p, 2 p + 1
      constexpr int v = 2 * decltype(p_c)::value, ks = v / 16, qt = (v / 8) % 2, e = v % 8, i = 8 * (ks % 2) + e;
      typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
      uint32_t w2 = __builtin_bit_cast(uint32_t, bf16x2{(__bf16)s[ks / 2][qt][i], (__bf16)s[ks / 2][qt][i + 1]});
      asm volatile("" : "+v"(w2));
      pf[ks][qt][e / 2] = w2;
    };
    float mx[2] = {-INFINITY, -INFINITY}, sum[2][2];
    auto vmax = [&](auto n_c) {
      constexpr int n = decltype(n_c)::value, t = n % 2, kt = (n / 2) % 2, i = 2 * (n / 4);
      mx[t] = fmaxf(fmaxf(mx[t], sn[kt][t][i]), sn[kt][t][i + 1]);
    };
    auto vsum = [&](auto v_c) {
      constexpr int v = decltype(v_c)::value, ks = v / 16, qt = (v / 8) % 2, i = 8 * (ks % 2) + v % 8, ch = v % 2;
      if constexpr (v < 16 && v % 8 < 2) sum[qt][ch] = s[ks / 2][qt][i];
      else {
        float x = sum[qt][ch] + s[ks / 2][qt][i];
        asm volatile("" : "+v"(x));
        sum[qt][ch] = x;
      }
    };
    constexpr int kHA = 2 * kSA, kHB = 2 * kSB;  // half steps
    using Plan = AttnPlan<kHA, kHB, kGA, kGB, 2 * kDma>;
    static constexpr Plan plan{};
    static_assert(plan.c[kHA] >= 8 && plan.c[kHA + kHB / 4] >= 16 && plan.c[kHA + kHB / 2] >= 24 &&
                      plan.c[kHA + 3 * (kHB / 4)] == 32, "a value product's probabilities are ready before it");
    static_assert(plan.x[kHA + kHB - 3] == 32, "maximum before the end");
    auto vec = [&](auto t_c) {
      constexpr int t = decltype(t_c)::value;
      if constexpr (Plan::dma(t) >= 0 && Plan::dma(t) < kDma) dma_k(j + 3, Plan::dma(t));
      if constexpr (Plan::dma(t) >= kDma) dma_v(j + 1, Plan::dma(t) - kDma);
      static_for<plan.c[t + 1], plan.c[t]>(vcvt);
      static_for<plan.e[t + 1], plan.e[t]>(vexp);
      static_for<plan.f[t + 1], plan.f[t]>(vfma);
      static_for<plan.x[t + 1], plan.x[t]>(vmax);
      static_for<plan.s[t + 1], plan.s[t]>(vsum);
      if constexpr (t == kHA + kHB - 3) {
        mx[0] = half_max(mx[0]);
        mx[1] = half_max(mx[1]);
      }
    };
    static_for<4>([&](auto g_c) {
      constexpr int g = decltype(g_c)::value;
      if constexpr (g == 3) {
        dma_barrier();  // the last fragments of K are in registers
      } else {
        __builtin_amdgcn_s_waitcnt(0xC07F);  // lgkmcnt(0): this group's fragments
      }
      static_for<2 * kGA>([&](auto u_c) {
        constexpr int u = decltype(u_c)::value, hs = 2 * kGA * g + u, f = hs / 2, c = f / 2, kt = f % 2, qt = u % 2;
        f32x16 z;
#pragma unroll
        for (int i = 0; i < 16; ++i) z[i] = 0.f;
        sn[kt][qt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fr[g % 2][u / 2], qf[qt][c], c == 0 ? z : sn[kt][qt], 0, 0, 0);
        if constexpr (g == 3 && u < kGB) fr[0][u] = vfrag(VP{}, u_c);
        if constexpr (g < 3 && u < kGA) fr[(g + 1) % 2][u] = kfrag(KP{}, std::integral_constant<int, kGA * (g + 1) + u>{});
        vec(std::integral_constant<int, hs>{});
        __builtin_amdgcn_sched_barrier(0);
      });
    });
    if (j + 2 == n_w) mask(sn);  // tile j + 1 is the wave's last: its diagonal
    __builtin_amdgcn_sched_barrier(0);
    static_for<4>([&](auto g_c) {
      constexpr int g = decltype(g_c)::value;
      __builtin_amdgcn_s_waitcnt(0xC07F);
      static_for<2 * kGB>([&](auto u_c) {
        constexpr int u = decltype(u_c)::value, hs = 2 * kGB * g + u, qt = u % 2, dt = u / 2;
        mfma_acc(acc[dt][qt], fr[g % 2][dt], pf[g][qt]);
        if constexpr (g < 3 && u < kGB) fr[(g + 1) % 2][u] = vfrag(VP{}, std::integral_constant<int, kGB * (g + 1) + u>{});
        if constexpr (g == 3 && u < kGA) fr[0][u] = kfrag(VP{}, u_c);  // tile j + 2's K has the parity of V
        vec(std::integral_constant<int, kHA + hs>{});
        __builtin_amdgcn_sched_barrier(0);
      });
    });
#pragma unroll
    for (int qt = 0; qt < 2; ++qt) l[qt] += sum[qt][0] + sum[qt][1];
    if (j + 1 < n_w) {
      // The reference stays until a logit passes it by 2^8: the exponentials
      // stay far from overflow and the sums are rescaled only then.
      const float r0 = mx[0] * c2, r1 = mx[1] * c2;
      if (__ballot(r0 > m[0] + 8.f || r1 > m[1] + 8.f)) {
        settle(acc);
        const float rr[2] = {r0, r1};
#pragma unroll
        for (int qt = 0; qt < 2; ++qt) {
          const float mn = fmaxf(m[qt], rr[qt]);
          const float alpha = __builtin_amdgcn_exp2f(m[qt] - mn);
          m[qt] = mn;
          l[qt] *= alpha;
#pragma unroll
          for (int dt = 0; dt < kDt; ++dt) acc[dt][qt] *= alpha;
        }
        settle(acc);
      }
    }
  };

  // Tile 0's logits and reference.
  dma_barrier();
  if (n_w > 0) {
    static_for<kSA>([&](auto f_c) {
      constexpr int f = decltype(f_c)::value, kt = f % 2, c = f / 2;
      const bf16x8 kf = kfrag(std::integral_constant<int, 0>{}, f_c);
#pragma unroll
      for (int qt = 0; qt < 2; ++qt) {
        f32x16 z;
#pragma unroll
        for (int i = 0; i < 16; ++i) z[i] = 0.f;
        s0[kt][qt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf, qf[qt][c], c == 0 ? z : s0[kt][qt], 0, 0, 0);
      }
    });
    if (n_w == 1) mask(s0);
#pragma unroll
    for (int qt = 0; qt < 2; ++qt) {
      float mx = -INFINITY;
#pragma unroll
      for (int kt = 0; kt < 2; ++kt)
#pragma unroll
        for (int i = 0; i < 16; ++i) mx = fmaxf(mx, s0[kt][qt][i]);
      m[qt] = half_max(mx) * c2;
    }
    static_for<kGA>([&](auto i_c) { fr[0][decltype(i_c)::value] = kfrag(std::integral_constant<int, 1>{}, i_c); });
  }
  middle(-1);
  using P0 = std::integral_constant<int, 0>;
  using P1 = std::integral_constant<int, 1>;
  if (n_w > 0) {
    for (int j = 0; j < n_w; j += 2) {
      step(P0{}, s0, s1, j);
      if (j + 1 < n_w) step(P1{}, s1, s0, j + 1);
    }
  }
  settle(acc);
  for (int j = n_w; j < n_kv; ++j) middle(j);  // the other waves' tiles

  // Normalise and store: lane (hl, m32) holds O[row][32 dt + 8 (i / 4) + 4 hl + i % 4].
#pragma unroll
  for (int qt = 0; qt < 2; ++qt) {
    const int qi = qw0 + 32 * qt + m32;
    auto p = __builtin_amdgcn_permlane32_swap(__float_as_uint(l[qt]), __float_as_uint(l[qt]), false, false);
    const float lt = __uint_as_float(p[0]) + __uint_as_float(p[1]);
    if (qi < L) {
      const float inv = 1.f / lt;
      __bf16* orow = a.out + ((int64_t)bhq * L + qi) * D;
#pragma unroll
      for (int dt = 0; dt < kDt; ++dt)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const f32x16& o = acc[dt][qt];
          const bf16x4 x = {(__bf16)(o[4 * i] * inv), (__bf16)(o[4 * i + 1] * inv), (__bf16)(o[4 * i + 2] * inv),
                            (__bf16)(o[4 * i + 3] * inv)};
          *reinterpret_cast<bf16x4*>(orow + 32 * dt + 8 * i + 4 * hl) = x;
        }
      if (hl == 0) a.lse[(int64_t)bhq * L + qi] = (m[qt] + __log2f(lt)) * 0.69314718055994531f;
    }
  }
}

// lse_proxy[b, hq, p] = lse[b, hq, pos[p]] (NaN for a position outside
// [0, L), which a device copy that disagrees with the validated host
// positions could hold; nothing outside the head is read).
__global__ __launch_bounds__(256) void lse_gather_kernel(const float* lse, const int32_t* pos, int L, int P,
                                                         int64_t n, float* out) {
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (i >= n) return;
  const int64_t bh = i / P;
  const int j = pos[i - bh * P];
  out[i] = j >= 0 && j < L ? lse[bh * L + j] : __builtin_nanf("");
}

template <int D, int NW>
void launch_attention_t(AttnLaunch a, hipStream_t stream) {
  const int heads = a.B * a.H * a.G;
  a.n_tiles = (a.L + 64 * NW - 1) / (64 * NW);
  a.heads_x = heads / 8;
  // Heads whose tiles run at the same time on an XCD: as many as have K and V
  // within its 4 MB L2 (the query heads of one K/V head count once).
  const int64_t kv = (int64_t)a.L * D * 4;
  a.group = (int)std::max<int64_t>(1, std::min<int64_t>(a.heads_x, a.G * std::max<int64_t>(1, (3 << 20) / kv)));
  const int64_t slots = (int64_t)a.heads_x * a.n_tiles + ((int64_t)(heads - 8 * a.heads_x) * a.n_tiles + 7) / 8;
  hipLaunchKernelGGL((attn_fwd_kernel<D, NW>), dim3((unsigned)(8 * slots)), dim3(64 * NW), 0, stream, a);
}

}  // namespace

hipError_t launch_attention(const AttnLaunch& a, int D, const int32_t* pos, int P, float* lse_proxy,
                            hipStream_t stream) {
  // 256 rows per work-group read K and V half as often as 128; with fewer
  // than 64 such work-groups (a quarter of the CUs) the finer tiles are dealt
  // more evenly: 8 heads of 1024 rows 30.5 against 31.9 us, 9 heads of 3854
  // (144 work-groups) 91.5 against 89.1, 32 heads of 32k 7.47 against 6.98 ms.
  const bool wide = (int64_t)a.B * a.H * a.G * ((a.L + 255) / 256) >= 64;
  if (D == 128) {
    if (wide) launch_attention_t<128, 4>(a, stream);
    else launch_attention_t<128, 2>(a, stream);
  } else {
    if (wide) launch_attention_t<64, 4>(a, stream);
    else launch_attention_t<64, 2>(a, stream);
  }
  hipError_t e = hipGetLastError();
  if (e != hipSuccess || !lse_proxy) return e;
  const int64_t n = (int64_t)a.B * a.H * a.G * P;
  hipLaunchKernelGGL(lse_gather_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, stream, a.lse, pos,
                     a.L, P, n, lse_proxy);
  return hipGetLastError();
}

}  // namespace nacl
