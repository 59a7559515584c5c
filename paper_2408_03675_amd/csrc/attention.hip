// Causal attention of the prefill with each query row's log-sum-exp: the
// forward pass of FlashAttention-2 that Appendix A.7 reuses, whose
// log-sum-exp lets the proxy-token score run as the single column reduction
// of Algorithm 2 (nacl_score's lse argument).  bf16 Q, K, V and output,
// fp32 accumulation, head dim 64 or 128, grouped query heads.
//
// Two kernels (launch_attention chooses): waves of 32 query rows, and for long
// heads of 128 waves of 64.  Both stream a head's keys in tiles of 64, with
// keys as the rows of S^T = K Q^T, so that a lane owns one query row per tile
// and the softmax statistics are per-lane scalars, and take the exponentials
// of a tile against the exact maximum of the row up to and with that tile: the
// largest probability is 1, which bf16 holds without error.  (A reference that
// stayed until a logit passed it by 2^8 spared most rescales of the output but
// rounded that probability like any other: the output's error against 64 bits
// grew from 1.86e-3 to 2.18e-3 with logits of standard deviation 2.)

#include <type_traits>

#include "device_common.h"
#include "internal.h"

namespace nacl {

namespace {

constexpr int kAttnKeys = 64;   // keys per tile
constexpr int kRsrcWord3 = 0x00020000;

typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));

// The query head and query tile of this work-group; false: none.  Work-groups
// are dealt to the 8 XCDs in turn: XCD x takes its share of the tiles of the
// heads that 8 does not divide, then heads x * heads_x .. in groups of `group`
// heads (whose K and V share its L2), the longest tiles of a group first, so
// that the last ones to start are short.  Against heads one after the other on
// each XCD (waves of 32 rows): 64 heads of 1536 rows of 128 83 -> 59 us, 128
// of 1024 82 -> 65, 32 of 2048 rows of 64 50 -> 40; the same where work-groups
// number fewer than the CUs.
__device__ __forceinline__ bool head_tile(const AttnLaunch& a, int& bhq, int& tile) {
  const int xcd = blockIdx.x & 7, n_heads = a.B * a.H * a.G, rest0 = 8 * a.heads_x, n_rest = n_heads - rest0;
  const int rest = (n_rest * a.n_tiles - xcd + 7) / 8;  // of the remaining heads' tiles
  int slot = blockIdx.x >> 3;
  if (slot < rest) {
    const int u = 8 * slot + xcd;
    tile = a.n_tiles - 1 - u / n_rest;
    bhq = rest0 + u % n_rest;
  } else {
    slot -= rest;
    if (slot >= a.heads_x * a.n_tiles) return false;
    const int g0 = slot / (a.group * a.n_tiles) * a.group, gn = min(a.group, a.heads_x - g0);
    const int i = slot - g0 * a.n_tiles;
    tile = a.n_tiles - 1 - i / gn;
    bhq = xcd * a.heads_x + g0 + i % gn;
  }
  bhq = __builtin_amdgcn_readfirstlane(bhq);
  tile = __builtin_amdgcn_readfirstlane(tile);
  return true;
}

// ---------------------------------------------------------------------------
// Waves of 32 query rows.  One work-group of 4 waves takes 128 consecutive
// query rows of one query head; wave w holds rows 32w .. 32w + 31 (two 16-row
// MFMA tiles) in registers:
//   S^T = K Q^T      v_mfma_f32_16x16x32_bf16, keys as MFMA rows, so lane
//                    (g, r) holds keys 4g .. 4g + 3 of each 16-key block for
//                    query r: every lane owns one query per MFMA tile, and
//                    the running maximum, sum and output rescale are
//                    per-lane scalars (the four lane groups agree on the
//                    maximum through two permlane swaps)
//   O^T += V^T P^T   the exponentials P in bf16 as the B operand straight
//                    from the S^T registers (lane (g, r) supplies keys
//                    4g .. 4g + 3 of two 16-key blocks, a permutation of the
//                    contraction that the A operand repeats), V^T from LDS.
// K and V tiles are loaded into registers one tile ahead and written into
// the other half of a double buffer in LDS after the tile in hand is done,
// so one barrier per tile separates the stages: K rows with their 16-byte
// chunks XOR-swizzled (the 16 rows of a fragment read hit distinct banks),
// V transposed (V^T[d][key], each lane's 8 keys of a fragment in one
// XOR-swizzled 16-byte chunk).  Two waves per SIMD; the fragment reads of 32
// rows take 128 LDS bytes per cycle at the matrix rate, all the LDS delivers,
// which bounds it where the chip is full.
constexpr int kAttnThreads = 256;
constexpr int kAttnRows = 128;  // query rows per work-group

__device__ __forceinline__ void attn_barrier() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }
// s_waitcnt vmcnt(0) (expcnt and lgkmcnt fields at their maxima), as an
// instruction the compiler's own wait counting sees.
__device__ __forceinline__ void wait_vm_all() { __builtin_amdgcn_s_waitcnt(0x0F70); }

// Maximum / sum over the four lane groups (lanes r, r + 16, r + 32, r + 48).
__device__ __forceinline__ float group_max(float x) {
  auto a = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  x = fmaxf(__uint_as_float(a[0]), __uint_as_float(a[1]));
  auto b = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return fmaxf(__uint_as_float(b[0]), __uint_as_float(b[1]));
}
__device__ __forceinline__ float group_sum(float x) {
  auto a = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  x = __uint_as_float(a[0]) + __uint_as_float(a[1]);
  auto b = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return __uint_as_float(b[0]) + __uint_as_float(b[1]);
}

template <int D>
__global__ __launch_bounds__(kAttnThreads, 2) void attn_fwd_kernel(AttnLaunch a) {
  constexpr int kRowBytes = D * 2;         // one K or V row
  constexpr int kChunks = kRowBytes / 16;  // 16-byte chunks per row
  constexpr int kSwz = kChunks - 1;
  constexpr int kKb = D / 32;              // contraction steps of S^T
  constexpr int kDt = D / 16;              // 16-wide d tiles of O^T
  constexpr int kTileBytes = kAttnKeys * kRowBytes;
  constexpr int kKUnits = kAttnKeys * kChunks / kAttnThreads;        // 16-byte K chunks per thread
  constexpr int kVUnits = (kAttnKeys / 2) * kChunks / kAttnThreads;  // (key pair, chunk) per thread
  static_assert(kKUnits >= 1 && kVUnits >= 1, "tile shape");

  __shared__ __attribute__((aligned(16))) unsigned char kbuf[2][kTileBytes];  // K rows, chunks swizzled
  __shared__ __attribute__((aligned(16))) unsigned char vbuf[2][kTileBytes];  // V^T[d][64 keys]

  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int g = lane >> 4, r = lane & 15;

  int bhq, tile;
  if (!head_tile(a, bhq, tile)) return;
  const int Hq = a.H * a.G;
  const int b = bhq / Hq, hq = bhq - b * Hq, h = hq / a.G;
  const int L = a.L;
  const int q0 = tile * kAttnRows;
  const int qw0 = q0 + 32 * wave;
  const int n_kv = (min(q0 + kAttnRows, L) + kAttnKeys - 1) / kAttnKeys;

  const __bf16* qh = a.q + (int64_t)b * a.qs[0] + (int64_t)hq * a.qs[1];
  const __bf16* kh = a.k + (int64_t)b * a.ks[0] + (int64_t)h * a.ks[1];
  const __bf16* vh = a.v + (int64_t)b * a.vs[0] + (int64_t)h * a.vs[1];
  const uint32_t qrow = (uint32_t)a.qs[2] * 2u, krow = (uint32_t)a.ks[2] * 2u, vrow = (uint32_t)a.vs[2] * 2u;
  // Rows at or past L read as zeros through the descriptors' ranges.
  const __amdgpu_buffer_rsrc_t qr = __builtin_amdgcn_make_buffer_rsrc(const_cast<__bf16*>(qh), (short)0,
                                                                      (int)((uint32_t)L * qrow), kRsrcWord3);
  const __amdgpu_buffer_rsrc_t kr = __builtin_amdgcn_make_buffer_rsrc(const_cast<__bf16*>(kh), (short)0,
                                                                      (int)((uint32_t)L * krow), kRsrcWord3);
  const __amdgpu_buffer_rsrc_t vr = __builtin_amdgcn_make_buffer_rsrc(const_cast<__bf16*>(vh), (short)0,
                                                                      (int)((uint32_t)L * vrow), kRsrcWord3);

  // Q fragments (B operand of S^T): query row qw0 + 16 qt + r, d = 32 kb + 8 g .. + 7.
  bf16x8 qf[2][kKb];
#pragma unroll
  for (int qt = 0; qt < 2; ++qt)
#pragma unroll
    for (int kb = 0; kb < kKb; ++kb)
      qf[qt][kb] = __builtin_bit_cast(
          bf16x8, __builtin_amdgcn_raw_buffer_load_b128(qr, (uint32_t)(qw0 + 16 * qt + r) * qrow + (uint32_t)(64 * kb + 16 * g),
                                                        0, 0));

  // K units: (row u / kChunks, chunk u mod kChunks) for u = tid + 256 s:
  // 16 lanes read one row's 256 contiguous bytes (D = 128); the chunk goes
  // to position chunk ^ (row & kSwz) of its LDS row.
  u32x4 kreg[kKUnits];
  auto load_k = [&](int j) {
#pragma unroll
    for (int s = 0; s < kKUnits; ++s) {
      const int u = tid + kAttnThreads * s;
      kreg[s] = __builtin_amdgcn_raw_buffer_load_b128(
          kr, (uint32_t)(j * kAttnKeys + u / kChunks) * krow + (uint32_t)(u % kChunks) * 16u, 0, 0);
    }
  };
  auto write_k = [&](int buf) {
#pragma unroll
    for (int s = 0; s < kKUnits; ++s) {
      const int u = tid + kAttnThreads * s;
      const int row = u / kChunks;
      *reinterpret_cast<u32x4*>(kbuf[buf] + row * kRowBytes + (((u % kChunks) ^ (row & kSwz)) * 16)) = kreg[s];
    }
  };
  // V units: (key pair kp = tid mod 32, chunk c = tid / 32 + 8 u): rows 2 kp
  // and 2 kp + 1, d = 8 c .. 8 c + 7.
  const int kp = tid & 31;
  u32x4 vreg[kVUnits][2];
  auto load_v = [&](int j) {
#pragma unroll
    for (int u = 0; u < kVUnits; ++u) {
      const int c = (tid >> 5) + 8 * u;
#pragma unroll
      for (int e = 0; e < 2; ++e)
        vreg[u][e] = __builtin_amdgcn_raw_buffer_load_b128(
            vr, (uint32_t)(j * kAttnKeys + 2 * kp + e) * vrow + (uint32_t)c * 16u, 0, 0);
    }
  };
  // V^T row d (128 bytes) holds the tile's 64 keys permuted so that the 8
  // keys lane group g contributes to contraction block kb2 (keys 32 kb2 +
  // 4 g .. + 3 and 32 kb2 + 16 + 4 g .. + 3) form 16-byte chunk 4 kb2 + g,
  // stored at chunk position (4 kb2 + g) ^ ((d >> 1) & 7): the 16 rows one
  // fragment read touches then cover every bank once per row parity.
  // Per V unit: the byte offset of d = 8 c + 2 h (h = 0..3) in its V^T row
  // pair, chunk swizzle included; d = 8 c + 2 h + 1 is the next row.
  uint32_t vto[kVUnits][4];
  {
    // keys 2 kp, 2 kp + 1: block kp >> 4, half (kp >> 3) & 1, group (kp >> 1) & 3,
    // the first of them at 2 (kp & 1) within its 4 keys
    const int c16 = 4 * (kp >> 4) + ((kp >> 1) & 3);
    const int dw = 2 * ((kp >> 3) & 1) + (kp & 1);  // dword within the chunk
#pragma unroll
    for (int u = 0; u < kVUnits; ++u) {
      const int c = (tid >> 5) + 8 * u;
#pragma unroll
      for (int h = 0; h < 4; ++h) {
        const int d = 8 * c + 2 * h;
        vto[u][h] = (uint32_t)(d * 128 + ((c16 ^ ((d >> 1) & 7)) * 16) + dw * 4);
      }
    }
  }
  auto write_vt = [&](int buf) {
#pragma unroll
    for (int u = 0; u < kVUnits; ++u) {
#pragma unroll
      for (int jj = 0; jj < 8; ++jj) {
        // bf16 jj of rows 2 kp (low half) and 2 kp + 1 (high half): bytes
        // 2 (jj mod 2) .. + 1 of word jj / 2 of each
        const uint32_t w = __builtin_amdgcn_perm(vreg[u][1][jj >> 1], vreg[u][0][jj >> 1],
                                                 (jj & 1) ? 0x07060302u : 0x05040100u);
        *reinterpret_cast<uint32_t*>(vbuf[buf] + vto[u][jj >> 1] + (jj & 1) * 128) = w;
      }
    }
  };

  const float c2 = a.c2;
  f32x4 acc[2][kDt];
#pragma unroll
  for (int qt = 0; qt < 2; ++qt)
#pragma unroll
    for (int dt = 0; dt < kDt; ++dt) acc[qt][dt] = f32x4{0.f, 0.f, 0.f, 0.f};
  float m[2] = {-INFINITY, -INFINITY}, l[2] = {0.f, 0.f};

  load_k(0);
  load_v(0);
  wait_vm_all();
  write_k(0);
  write_vt(0);
  if (n_kv > 1) {
    load_k(1);
    load_v(1);
  }
  attn_barrier();

  for (int j = 0; j < n_kv; ++j) {
    const int buf = j & 1;
    const int key0 = j * kAttnKeys;
    if (key0 <= qw0 + 31) {  // some key of the tile is visible to a row of this wave
      const unsigned char* kt_base = kbuf[buf];
      const unsigned char* vt_base = vbuf[buf];
      // S^T tiles: kt (16 keys) x qt (16 queries).
      f32x4 s[4][2];
#pragma unroll
      for (int kt = 0; kt < 4; ++kt) {
        const int row = 16 * kt + r;
        bf16x8 kf[kKb];
#pragma unroll
        for (int kb = 0; kb < kKb; ++kb)
          kf[kb] = __builtin_bit_cast(
              bf16x8, *reinterpret_cast<const u32x4*>(kt_base + row * kRowBytes + (((4 * kb + g) ^ (row & kSwz)) * 16)));
#pragma unroll
        for (int qt = 0; qt < 2; ++qt) {
          f32x4 t = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
          for (int kb = 0; kb < kKb; ++kb) t = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kf[kb], qf[qt][kb], t, 0, 0, 0);
          s[kt][qt] = t;
        }
      }
      // Value fragment (A operand of O^T): V^T row d = 16 dt + r, chunk 4 kb2 + g.
      auto vfrag = [&](int dt, int kb2) {
        const int d = 16 * dt + r;
        return __builtin_bit_cast(
            bf16x8, *reinterpret_cast<const u32x4*>(vt_base + d * 128 + (((4 * kb2 + g) ^ ((d >> 1) & 7)) * 16)));
      };
      // The first d tile's value fragments are read before the exponentials.
      bf16x8 vcur[2] = {vfrag(0, 0), vfrag(0, 1)};
      __builtin_amdgcn_sched_barrier(0);
      const bool masked = key0 + kAttnKeys - 1 > qw0;
      bf16x8 pf[2][2];  // [qt][kb2]
#pragma unroll
      for (int qt = 0; qt < 2; ++qt) {
        const int qi = qw0 + 16 * qt + r;
        if (masked) {
          // key key0 + 16 kt + 4 g + i is past row qi iff 16 kt + i > lim
          const int lim = qi - key0 - 4 * g;
#pragma unroll
          for (int kt = 0; kt < 4; ++kt)
#pragma unroll
            for (int i = 0; i < 4; ++i)
              if (16 * kt + i > lim) s[kt][qt][i] = -INFINITY;
        }
        // The scale is positive, so the largest logit is the scaled largest
        // raw product; each exponent is then one FMA.
        float mx = -INFINITY;
#pragma unroll
        for (int kt = 0; kt < 4; ++kt)
#pragma unroll
          for (int i = 0; i < 4; ++i) mx = fmaxf(mx, s[kt][qt][i]);
        mx = group_max(mx);
        const float mn = fmaxf(m[qt], mx * c2);
        const float alpha = __builtin_amdgcn_exp2f(m[qt] - mn);
        m[qt] = mn;
        float x[4][4];
        float sum = 0.f;
#pragma unroll
        for (int kt = 0; kt < 4; ++kt)
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            x[kt][i] = __builtin_amdgcn_exp2f(__builtin_fmaf(s[kt][qt][i], c2, -mn));
            sum += x[kt][i];
          }
        l[qt] = l[qt] * alpha + sum;
        // Rescale only when some row of the wave raised its maximum.
        if (__ballot(alpha != 1.f)) {
#pragma unroll
          for (int dt = 0; dt < kDt; ++dt) acc[qt][dt] *= alpha;
        }
#pragma unroll
        for (int kb2 = 0; kb2 < 2; ++kb2)
          pf[qt][kb2] = bf16x8{(__bf16)x[2 * kb2][0], (__bf16)x[2 * kb2][1], (__bf16)x[2 * kb2][2],
                               (__bf16)x[2 * kb2][3], (__bf16)x[2 * kb2 + 1][0], (__bf16)x[2 * kb2 + 1][1],
                               (__bf16)x[2 * kb2 + 1][2], (__bf16)x[2 * kb2 + 1][3]};
      }
      // O^T += V^T P^T; the reads of d tile dt + 1 are issued before the
      // products of d tile dt.
#pragma unroll
      for (int dt = 0; dt < kDt; ++dt) {
        bf16x8 vnxt[2];
        if (dt + 1 < kDt) {
          vnxt[0] = vfrag(dt + 1, 0);
          vnxt[1] = vfrag(dt + 1, 1);
        }
#pragma unroll
        for (int kb2 = 0; kb2 < 2; ++kb2)
#pragma unroll
          for (int qt = 0; qt < 2; ++qt)
            acc[qt][dt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(vcur[kb2], pf[qt][kb2], acc[qt][dt], 0, 0, 0);
        if (dt + 1 < kDt) {
          __builtin_amdgcn_sched_group_barrier(0x100, 2, 0);  // the two reads
          __builtin_amdgcn_sched_group_barrier(0x008, 4, 0);  // then the four products
          vcur[0] = vnxt[0];
          vcur[1] = vnxt[1];
        }
      }
    }
    if (j + 1 < n_kv) {
      wait_vm_all();  // this thread's K and V rows of tile j + 1
      write_k(buf ^ 1);
      write_vt(buf ^ 1);
    }
    attn_barrier();  // tile j read by every wave; tile j + 1 written
    if (j + 2 < n_kv) {
      load_k(j + 2);
      load_v(j + 2);
    }
  }

  // Normalise and store: lane (g, r) holds O[row][16 dt + 4 g .. + 3].
#pragma unroll
  for (int qt = 0; qt < 2; ++qt) {
    const int qi = qw0 + 16 * qt + r;
    const float lt = group_sum(l[qt]);
    if (qi < L) {
      const float inv = 1.f / lt;
      __bf16* orow = a.out + ((int64_t)bhq * L + qi) * D;
#pragma unroll
      for (int dt = 0; dt < kDt; ++dt) {
        const bf16x4 o = {(__bf16)(acc[qt][dt][0] * inv), (__bf16)(acc[qt][dt][1] * inv),
                          (__bf16)(acc[qt][dt][2] * inv), (__bf16)(acc[qt][dt][3] * inv)};
        *reinterpret_cast<bf16x4*>(orow + 16 * dt + 4 * g) = o;
      }
      if (g == 0) a.lse[(int64_t)bhq * L + qi] = (m[qt] + __log2f(lt)) * 0.69314718055994531f;
    }
  }
}

// ---------------------------------------------------------------------------
// Waves of 64 query rows (head dim 128): a work-group of 4 waves takes 256
// consecutive rows of one query head, each wave two 32-row MFMA tiles:
//   S^T = K Q^T   v_mfma_f32_32x32x16_bf16, keys as MFMA rows: lane (hl, r)
//                 holds keys 8 i + 4 hl .. + 3 of each 32-key block for query r
//                 (the two lane halves agree through one permlane swap)
//   O += P V      the exponentials P in bf16 as the A operand straight from the
//                 S^T registers, V by transposing LDS reads of the same keys (a
//                 permutation of the contraction); lane (hl, d) holds rows
//                 8 (i / 4) + 4 hl + i % 4 of column d in accumulator register i.
//
// What bounds it, and why it looks like this.  Per 64-key tile a wave has 64
// MFMAs (32 cycles each) and, for each of a lane's 64 logits, an FMA, an
// exponential, an addition and half a maximum and conversion.
// - 64 rows per wave: an LDS fragment then serves two MFMAs of 32 cycles, 64
//   bytes per cycle and CU where 32 rows take 128.  It takes 64 + 128
//   accumulation registers for Q and O and about 250 vector registers for two
//   tiles of logits: one wave per SIMD.
// - With one wave per SIMD, matrix and vector work overlap only within the
//   wave: a software pipeline runs the logits of tile j + 1 beside the
//   exponentials of tile j, and the value products of tile j beside its row
//   sums and the maxima of tile j + 1.  AttnPlan deals the vector operations
//   to half steps of one MFMA each, equal in issue cycles, and
//   sched_barriers keep them there.
// - A tile that raises a row's maximum rescales that row's output: O's rows lie
//   along the registers, so a row and its partner in the other lane half are
//   four accumulator registers.  In the first tiles nearly every row of a wave
//   rises, later few do.  32 heads of 32k rows: 6.9 ms without any rescale, 7.5
//   as it is, 8.8 if all 64 rows are rescaled when one rises.
// - K and V go from memory to LDS by DMA (buffer loads with the lds flag),
//   two tiles of each, spread over the half steps; the loop has one barrier
//   per tile, in the middle: K is loaded two tiles ahead of its use and V
//   one, K's last fragments are in registers when the barrier is passed.
// 128 heads of 32k rows: 34.7 ms by waves of 32 rows, 29.8 here (1.18 PFLOP/s; a
// plain bf16 product of 16384^3 reaches 1.37 on this part).

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
// the next one; the kernel waits for them itself (dma_barrier).
// (A vector instruction that writes a scalar register, as a spilled one's
// reload does, has to be five wait states ahead of a load that reads it: two
// instructions and three waits.  M0 is one of the compiler's own registers; it
// is told of the write all the same.)
#pragma clang diagnostic push
#pragma clang diagnostic ignored "-Winline-asm"
__device__ __forceinline__ void dma_1k(u32x4 rsrc, uint32_t voff, uint32_t off, uint32_t lds) {
  uint32_t t;
  asm volatile("s_mov_b32 m0, %1\n\tv_add_u32 %0, %2, %3\n\ts_nop 2\n\tbuffer_load_dwordx4 %0, %4, 0 offen lds"
               : "=&v"(t)
               : "s"(lds), "s"(off), "v"(voff), "s"(rsrc)
               : "memory", "m0");
}
#pragma clang diagnostic pop
// Every DMA of this wave and every LDS read it issued has completed, then
// the work-group's barrier.
__device__ __forceinline__ void dma_barrier() {
  asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier" ::: "memory");
}

typedef float f32x16 __attribute__((ext_vector_type(16)));

// acc += A B on the accumulation registers, where the output stays so that the
// vector registers hold two tiles of logits.  The compiler does not know an
// asm block's wait states: whatever else touches an accumulator does so after
// settle() or 18 wait states of other MFMAs, and an operand written by a vector
// instruction is written at least two instructions before (a tile's
// probabilities: at least one half step).
__device__ __forceinline__ void mfma_acc(f32x16& acc, u32x4 fa, bf16x8 fb) {
  asm volatile("v_mfma_f32_32x32x16_bf16 %0, %1, %2, %0" : "+a"(acc) : "v"(fa), "v"(fb));
}
// Register I of accumulator N, read and written where it is: in C the compiler
// copies the whole accumulator to vector registers and back, and to name one of
// its registers a block has to know which they are.
#define NACL_ACC(X) X(0, 0, 15) X(1, 16, 31) X(2, 32, 47) X(3, 48, 63) X(4, 64, 79) X(5, 80, 95) X(6, 96, 111) X(7, 112, 127)
template <int N, int I>
__device__ __forceinline__ float get_acc(f32x16& acc) {
  float t;
#define NACL_GET(M, LO, HI) \
  if constexpr (N == M) asm volatile("v_accvgpr_read_b32 %1, a[%2]" : "+{a[" #LO ":" #HI "]}"(acc), "=v"(t) : "n"(LO + I));
  NACL_ACC(NACL_GET)
#undef NACL_GET
  return t;
}
template <int N, int I>
__device__ __forceinline__ void set_acc(f32x16& acc, float t) {
#define NACL_SET(M, LO, HI) \
  if constexpr (N == M) asm volatile("v_accvgpr_write_b32 a[%2], %1" : "+{a[" #LO ":" #HI "]}"(acc) : "v"(t), "n"(LO + I));
  NACL_ACC(NACL_SET)
#undef NACL_SET
}
#undef NACL_ACC
// Nothing moves past here that touches an accumulator.  WAIT: every MFMA issued
// before has written its accumulator (32 wait states; a 32x32x16 needs 18).
// Otherwise four wait states, for MFMAs after a vector instruction's write.
template <bool WAIT>
__device__ __forceinline__ void settle(f32x16 (&acc)[4][2]) {
  if constexpr (WAIT) asm volatile("s_nop 15\n\ts_nop 15");
  asm volatile("s_nop 3"
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

constexpr int kLongWaves = 4;  // waves of 64 query rows per work-group

__global__ __launch_bounds__(64 * kLongWaves, 1) void attn_long_kernel(AttnLaunch a) {
  constexpr int D = 128, NW = kLongWaves;
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

  int bhq, tile;
  if (!head_tile(a, bhq, tile)) return;
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
  settle<true>(acc);
  float m[2] = {0.f, 0.f}, l[2] = {0.f, 0.f};  // row maxima (base-2 logits) and sums
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

  // Rows whose maximum the tile in hand raised, and their factors (1 for the
  // other rows of the 32): O takes them in the middle of the tile's step, all its
  // MFMAs of the tile before being done.
  uint32_t up[2] = {0u, 0u};
  float alpha[2] = {1.f, 1.f};
  auto rescale = [&]() __attribute__((always_inline)) {
    settle<false>(acc);
    static_for<2>([&](auto qt_c) __attribute__((always_inline)) {
      constexpr int qt = decltype(qt_c)::value;
      if (!up[qt]) return;
      // f[i]: the factor of row 16 i + n in lane n of each row of 16 lanes, of
      // row 16 i + n + 4 in the upper half.
      const uint32_t al = __float_as_uint(alpha[qt]);
      auto p = __builtin_amdgcn_permlane16_swap(al, al, false, false);
      int f[2];
#pragma unroll
      for (int i = 0; i < 2; ++i) f[i] = __builtin_amdgcn_update_dpp((int)p[i], (int)p[i], 0x104 /* row_shl:4 */, 0xC, 0xF, false);
      static_for<4>([&](auto g_c) __attribute__((always_inline)) {
        constexpr int g = decltype(g_c)::value;
        if (up[qt] & (0xFFu << (8 * g)))
          static_for<4>([&](auto e_c) __attribute__((always_inline)) {
            constexpr int e = decltype(e_c)::value, i = 4 * g + e;  // rows 8 g + e and 8 g + 4 + e
            if (up[qt] & (0x11u << (8 * g + e))) {
              float t[kDt];
              static_for<kDt>([&](auto dt_c) __attribute__((always_inline)) {
                constexpr int dt = decltype(dt_c)::value;
                t[dt] = get_acc<2 * dt + qt, i>(acc[dt][qt]);
              });
              // row_newbcast: lane n of each row of 16 lanes to all of them
              const float x = __uint_as_float((uint32_t)__builtin_amdgcn_update_dpp(0, f[g / 2], 0x150 + 8 * (g % 2) + e, 0xF, 0xF, true));
              static_for<kDt>([&](auto dt_c) __attribute__((always_inline)) {
                constexpr int dt = decltype(dt_c)::value;
                set_acc<2 * dt + qt, i>(acc[dt][qt], t[dt] * x);
              });
            }
          });
      });
    });
    settle<false>(acc);
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
    if (up[0] | up[1]) rescale();
    static_for<4>([&](auto g_c) {
      constexpr int g = decltype(g_c)::value;
      __builtin_amdgcn_s_waitcnt(0xC07F);
      static_for<2 * kGB>([&](auto u_c) {
        constexpr int u = decltype(u_c)::value, hs = 2 * kGB * g + u, qt = u % 2, dt = u / 2;
        mfma_acc(acc[dt][qt], pf[g][qt], fr[g % 2][dt]);
        if constexpr (g < 3 && u < kGB) fr[(g + 1) % 2][u] = vfrag(VP{}, std::integral_constant<int, kGB * (g + 1) + u>{});
        if constexpr (g == 3 && u < kGA) fr[0][u] = kfrag(VP{}, u_c);  // tile j + 2's K has the parity of V
        vec(std::integral_constant<int, kHA + hs>{});
        __builtin_amdgcn_sched_barrier(0);
      });
    });
#pragma unroll
    for (int qt = 0; qt < 2; ++qt) l[qt] += sum[qt][0] + sum[qt][1];
    if (j + 1 < n_w) {
      // The next tile's maxima (m stays where a logit is NaN: its exponential is).
      const float r[2] = {mx[0] * c2, mx[1] * c2};
#pragma unroll
      for (int qt = 0; qt < 2; ++qt) {
        up[qt] = (uint32_t)__ballot(r[qt] > m[qt]);
        if (up[qt]) {
          const float mn = fmaxf(m[qt], r[qt]);
          alpha[qt] = __builtin_amdgcn_exp2f(m[qt] - mn);
          m[qt] = mn;
          l[qt] *= alpha[qt];
        }
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
  settle<true>(acc);
  for (int j = n_w; j < n_kv; ++j) middle(j);  // the other waves' tiles
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // the loads past the last tile, which write zeros

  // Normalise and store: lane (hl, m32) holds O[8 (i / 4) + 4 hl + i % 4][32 dt
  // + m32].  Lanes 2 n and 2 n + 1 trade halves of two rows, so that each
  // stores two columns of one row.
#pragma unroll
  for (int qt = 0; qt < 2; ++qt) {
    auto p = __builtin_amdgcn_permlane32_swap(__float_as_uint(l[qt]), __float_as_uint(l[qt]), false, false);
    const float lt = __uint_as_float(p[0]) + __uint_as_float(p[1]);
    const float inv = 1.f / lt;
    const int qi = qw0 + 32 * qt + m32;
    if (qi < L && hl == 0) a.lse[(int64_t)bhq * L + qi] = (m[qt] + __log2f(lt)) * 0.69314718055994531f;
#pragma unroll
    for (int i = 0; i < 16; i += 2) {
      const int r = 8 * (i / 4) + 4 * hl + i % 4;
      const float inv0 = __shfl(inv, r), inv1 = __shfl(inv, r + 1);
      const int row = qw0 + 32 * qt + r + (lane & 1);
      __bf16* orow = a.out + ((int64_t)bhq * L + row) * D + (m32 & ~1);
#pragma unroll
      for (int dt = 0; dt < kDt; ++dt) {
        typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
        const uint32_t w = __builtin_bit_cast(uint32_t, bf16x2{(__bf16)(acc[dt][qt][i] * inv0), (__bf16)(acc[dt][qt][i + 1] * inv1)});
        const uint32_t o = (uint32_t)__builtin_amdgcn_mov_dpp((int)w, 0xB1, 0xF, 0xF, true);  // lane ^ 1
        const uint32_t x = lane & 1 ? __builtin_amdgcn_perm(w, o, 0x07060302u) : __builtin_amdgcn_perm(o, w, 0x05040100u);
        if (row < L) *reinterpret_cast<uint32_t*>(orow + 32 * dt) = x;
      }
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

// rows: query rows per work-group (of 256 threads).
template <class K>
void launch_attention_t(K kern, int D, int rows, AttnLaunch a, hipStream_t stream) {
  const int heads = a.B * a.H * a.G;
  a.n_tiles = (a.L + rows - 1) / rows;
  a.heads_x = heads / 8;
  // Heads whose tiles run at the same time on an XCD: as many as have K and V
  // within its 4 MB L2 (the query heads of one K/V head count once).
  const int64_t kv = (int64_t)a.L * D * 4;
  a.group = (int)std::max<int64_t>(1, std::min<int64_t>(a.heads_x, a.G * std::max<int64_t>(1, (3 << 20) / kv)));
  const int64_t slots = (int64_t)a.heads_x * a.n_tiles + ((int64_t)(heads - 8 * a.heads_x) * a.n_tiles + 7) / 8;
  hipLaunchKernelGGL(kern, dim3((unsigned)(8 * slots)), dim3(256), 0, stream, a);
}

}  // namespace

hipError_t launch_attention(const AttnLaunch& a, int D, const int32_t* pos, int P, float* lse_proxy,
                            hipStream_t stream) {
  // Waves of 64 rows where each CU gets a work-group of them and the rows are
  // long enough that rescales are few.  Rows of 128, waves of 32 against 64:
  // 32 heads of 2048 72 and 71 us, 4096 194 and 211, 6144 371 and 338, 16384
  // 2.27 and 1.99 ms; 8 heads of 6144 (192 work-groups) 158 and 167 us, 16384
  // 626 and 503; 2 heads of 32768 (256) 812 and 741.  Rows of 64 gain less
  // than 4 % where the chip is full and lose as much at 128 heads.
  const bool wide = D == 128 && a.L >= 6144 && (int64_t)a.B * a.H * a.G * ((a.L + 255) / 256) >= 256;
  if (wide) launch_attention_t(attn_long_kernel, D, 64 * kLongWaves, a, stream);
  else if (D == 128) launch_attention_t(attn_fwd_kernel<128>, D, kAttnRows, a, stream);
  else launch_attention_t(attn_fwd_kernel<64>, D, kAttnRows, a, stream);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess || !lse_proxy) return e;
  const int64_t n = (int64_t)a.B * a.H * a.G * P;
  hipLaunchKernelGGL(lse_gather_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, stream, a.lse, pos,
                     a.L, P, n, lse_proxy);
  return hipGetLastError();
}

}  // namespace nacl
