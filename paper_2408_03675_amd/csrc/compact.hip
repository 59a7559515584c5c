// Cache update K0, V0 <- K_S, V_S (NaCl Section 3, encoding-phase eviction):
// a row gather.  One thread moves one 16-byte vector: the lanes covering a
// row read it contiguously and write it to a contiguous output row, so both
// sides are coalesced.  K and V rows go to separate blocks (blockIdx.z), and
// with no loop every thread's load is in flight from its first instruction;
// many small blocks keep the whole chip issuing.  Rows are bit copies.
//
// Also here: the in-place form of the same update for a decode-time cache
// (Section 3, generation-phase eviction: the kept rows move to the front of
// each head's own rows), and the append of new decode steps' rows to the
// cache (Algorithm 1, generation phase).

#include "device_common.h"
#include "internal.h"

namespace nacl {

constexpr int kCompactThreads = 512;

// A keep index outside [0, L) gives a zero row and sets bit 2 of the health
// words (when the launch has them) instead of reading outside the head.
__device__ __forceinline__ void flag_bad_index(uint32_t* health) {
  if (health) {
    atomicOr(health, 4u);
    atomicOr(health + 1, 4u);
  }
}

// VPR: 16-byte vectors per row (D * element size / 16), a compile-time
// constant so the row and vector of a thread are shifts, not divisions.
template <int VPR>
__global__ __launch_bounds__(kCompactThreads) void compact_kernel(CompactLaunch a) {
  const int bh = blockIdx.y, b = bh / a.H, h = bh % a.H;
  constexpr int vpr = VPR;
  const int r = blockIdx.x * (kCompactThreads / vpr) + (int)threadIdx.x / vpr;
  if (r >= a.C) return;
  const int vec = threadIdx.x % vpr;
  const bool is_v = blockIdx.z != 0;
  const int64_t* st = is_v ? a.vs : a.ks;
  const int j = a.keep[(int64_t)bh * a.C + r];
  // The load is unconditional (an out-of-range index reads row 0 of the
  // head) so it issues as soon as the index arrives; its value is replaced
  // by zeros afterwards.
  const bool ok = (unsigned)j < (unsigned)a.L;
  const u32x4* src = static_cast<const u32x4*>(is_v ? a.v : a.k) + b * st[0] + h * st[1] +
                     (int64_t)(ok ? j : 0) * st[2] + vec;
  u32x4 x = __builtin_nontemporal_load(src);
  if (!ok) {
    x = u32x4{0u, 0u, 0u, 0u};
    if (vec == 0) flag_bad_index(a.health);
  }
  u32x4* dst = static_cast<u32x4*>(is_v ? a.v_out : a.k_out) + ((int64_t)bh * a.C + r) * vpr + vec;
  __builtin_nontemporal_store(x, dst);
}

// In place: row c of each head takes row keep[c] of the same head, in the
// input's own layout.  keep is strictly ascending, so keep[c] >= c and the
// rows a chunk of destinations [c0, c1) reads lie at or after c0: rows that
// no earlier chunk writes.  One work-group per (head, K or V, column slice)
// walks the chunks in order; inside a chunk every source is read (the barrier
// waits for the loads) before any destination is written, since a source of
// one row may be the destination of another row of the same chunk.  Rows with
// keep[c] == c stay where they are.
//
// A row's vectors keep their columns, so the order holds within each column
// by itself, and slices of SLICE vectors need no word between their
// work-groups: few heads still give enough loads in flight.  What bounds it is
// memory latency (a chunk's indices, its rows, then the stores) until every CU
// has work, and then HBM; a chunk's indices are read together, as a row's load
// behind its own index only would wait for them one by one.  Whole rows of 1024
// threads and indices one by one before, now (a call on buffers that are not in a
// cache): 4 heads of 131072 rows keeping 40000 (bf16, 128) 519 -> 140 us; 32
// heads, 32768 keeping 10000, 170 -> 74 (4.4 TB/s); 12 fp32 heads, 20001 keeping
// 7001, 199 -> 46; 128 heads, 16384 keeping 5000 (bf16, 64) 75 -> 71; 128 heads,
// 6617 keeping 6553, 181 -> 175.
constexpr int kInplaceVecs = 16;  // vectors per thread and chunk (all loads in flight at once)

constexpr int kInplaceThreads = 512;

template <int VPR, int SLICE>
__global__ __launch_bounds__(kInplaceThreads) void compact_inplace_kernel(CompactLaunch a) {
  static_assert(VPR % SLICE == 0 && kInplaceThreads % SLICE == 0);
  const int bh = blockIdx.x, b = bh / a.H, h = bh % a.H;
  const bool is_v = blockIdx.y % 2 != 0;
  const int col = (int)(blockIdx.y / 2) * SLICE;
  const int64_t* st = is_v ? a.vs : a.ks;
  u32x4* base = static_cast<u32x4*>(is_v ? a.v_out : a.k_out) + b * st[0] + h * st[1] + col + threadIdx.x % SLICE;
  constexpr int kRows = kInplaceThreads / SLICE;  // rows per vector of a thread
  const int32_t* keep = a.keep + (int64_t)bh * a.C;
  for (int c0 = 0; c0 < a.C; c0 += kRows * kInplaceVecs) {
    u32x4 x[kInplaceVecs];
    int dst[kInplaceVecs], src[kInplaceVecs];
#pragma unroll
    for (int u = 0; u < kInplaceVecs; ++u) src[u] = keep[min(c0 + u * kRows + (int)threadIdx.x / SLICE, a.C - 1)];
#pragma unroll
    for (int u = 0; u < kInplaceVecs; ++u) {
      const int r = c0 + u * kRows + (int)threadIdx.x / SLICE, j = src[u];
      const bool ok = (unsigned)j < (unsigned)a.L;
      dst[u] = r < a.C && j != r ? r : -1;
      x[u] = u32x4{0u, 0u, 0u, 0u};
      if (dst[u] >= 0 && ok) x[u] = base[(int64_t)j * st[2]];
      if (dst[u] >= 0 && !ok && col == 0 && threadIdx.x % SLICE == 0) flag_bad_index(a.health);
    }
    __syncthreads();
#pragma unroll
    for (int u = 0; u < kInplaceVecs; ++u)
      if (dst[u] >= 0) base[(int64_t)dst[u] * st[2]] = x[u];
  }
}

// Slot form of the in-place update (generation-phase eviction with a cache
// whose rows need not stay in token order): with S the ascending keep set of
// a head, the kept rows below C stay in their slots, and the kept rows at or
// past C (the movers, S[n_low..C)) fill the other slots below C (the free
// slots), both in ascending order.  Only the movers' rows are copied; their
// sources lie at or past C and their destinations below C, so no copy reads
// a row another one writes.  slots[c] = the old row slot c holds afterwards.
// Free slot number fi is f = fi + i*, i* the first i < n_low with
// S[i] - i > fi (S[i] - i free slots lie below S[i], a non-decreasing count),
// found by a binary search over S.  One work-group per head; VPR lanes per
// moved row (K and V).  A mover outside [C, L) (a keep list that is not an
// ascending set of rows) gives zero rows and sets bit 2 of the health words.
constexpr int kSlotThreads = 1024;
constexpr int kSlotLdsKeep = 16384;  // keep lists up to this long are searched in LDS

template <int VPR>
__global__ __launch_bounds__(kSlotThreads) void compact_slots_kernel(CompactLaunch a) {
  __shared__ int n_low_s;
  __shared__ int32_t keep_lds[kSlotLdsKeep];
  const int bh = blockIdx.x, b = bh / a.H, h = bh % a.H;
  const int32_t* Sg = a.keep + (int64_t)bh * a.C;
  int32_t* Y = a.slots + (int64_t)bh * a.C;
  u32x4* kb = static_cast<u32x4*>(a.k_out) + b * a.ks[0] + h * a.ks[1];
  u32x4* vb = static_cast<u32x4*>(a.v_out) + b * a.vs[0] + h * a.vs[1];
  constexpr int kRowsPerPass = kSlotThreads / VPR;
  const int vec = threadIdx.x % VPR;
  // The steps, over the keep list S (called with the LDS copy or with the
  // list in memory, each call on a pointer whose memory the compiler knows:
  // no generic pointer into LDS is formed).
  auto run = [&](const int32_t* S) {
    if (threadIdx.x == 0) n_low_s = a.C;
    __syncthreads();
    // The first entry at or past C (one writer when S ascends).
    for (int i = threadIdx.x; i < a.C; i += kSlotThreads)
      if (S[i] >= a.C && (i == 0 || S[i - 1] < a.C)) n_low_s = i;
    __syncthreads();
    const int n_low = n_low_s, n_move = a.C - n_low;
    for (int i = threadIdx.x; i < n_low; i += kSlotThreads) {
      const int r = S[i];
      if ((unsigned)r < (unsigned)a.C) Y[r] = r;  // a kept row below C keeps its slot
    }
    for (int fi0 = 0; fi0 < n_move; fi0 += kRowsPerPass) {
      const int fi = fi0 + (int)threadIdx.x / VPR;
      if (fi >= n_move) continue;
      int lo = 0, hi = n_low;
      while (lo < hi) {
        const int mid = (lo + hi) >> 1;
        if (S[mid] - mid > fi) hi = mid;
        else lo = mid + 1;
      }
      const int f = fi + lo;           // < n_move + n_low = C
      const int r = S[n_low + fi];     // the mover
      const bool ok = r >= a.C && r < a.L;
      if (vec == 0) {
        Y[f] = r;
        if (!ok) flag_bad_index(a.health);
      }
      const u32x4 z = {0u, 0u, 0u, 0u};
      const u32x4 xk = ok ? kb[(int64_t)r * a.ks[2] + vec] : z;
      const u32x4 xv = ok ? vb[(int64_t)r * a.vs[2] + vec] : z;
      kb[(int64_t)f * a.ks[2] + vec] = xk;
      vb[(int64_t)f * a.vs[2] + vec] = xv;
    }
  };
  // The binary searches read the keep list many times: from LDS when it fits.
  if (a.C <= kSlotLdsKeep) {
    for (int i = threadIdx.x; i < a.C; i += kSlotThreads) keep_lds[i] = Sg[i];
    run(keep_lds);
  } else {
    run(Sg);
  }
}

// Append: rows [row0, row0 + m) of every head of the cache take the m rows
// of k_new / v_new ([B, H, m, D] contiguous).
__global__ __launch_bounds__(kCompactThreads) void append_kernel(AppendLaunch a) {
  const int bh = blockIdx.y, b = bh / a.H, h = bh % a.H;
  const int vpr = a.row_vecs;
  const int r = blockIdx.x * (kCompactThreads / vpr) + (int)threadIdx.x / vpr;
  if (r >= a.m) return;
  const int vec = threadIdx.x % vpr;
  const bool is_v = blockIdx.z != 0;
  const int64_t* st = is_v ? a.vs : a.ks;
  const u32x4* src = static_cast<const u32x4*>(is_v ? a.v_new : a.k_new) + ((int64_t)bh * a.m + r) * vpr + vec;
  u32x4* dst = static_cast<u32x4*>(is_v ? a.v : a.k) + b * st[0] + h * st[1] + (int64_t)(a.row0 + r) * st[2] + vec;
  *dst = *src;
}

namespace {

template <int VPR>
hipError_t launch_compact_t(const CompactLaunch& a, hipStream_t stream) {
  if (a.in_place) {
    // Slices of 64 bytes while these give at most one work-group per CU (256);
    // beyond, a line shared by two work-groups costs more than the parallelism
    // gives (32 heads of 16 vectors a row, 256 work-groups: 66.6 us in 64-byte
    // slices, 80.9 in 128-byte ones; 128 heads 306 and 187), and work-groups take
    // whole rows: 128 heads of 2048 rows (bf16, 128) keeping 2000 54.5 us, in
    // 128-byte slices with 1024 threads 62.7; 1000 of 600 keeping 200 46 and 60,
    // fp32 88 and 116; 400 of 2000 keeping 1000 92 and 89.
    const int BH = a.B * a.H;
    if ((int64_t)2 * BH * (VPR / 4) <= 256)
      hipLaunchKernelGGL((compact_inplace_kernel<VPR, 4>), dim3(BH, 2 * (VPR / 4)), dim3(kInplaceThreads), 0, stream, a);
    else
      hipLaunchKernelGGL((compact_inplace_kernel<VPR, VPR>), dim3(BH, 2), dim3(kInplaceThreads), 0, stream, a);
    return hipGetLastError();
  }
  constexpr int rows_per_block = kCompactThreads / VPR;
  dim3 grid((a.C + rows_per_block - 1) / rows_per_block, a.B * a.H, 2);
  hipLaunchKernelGGL(compact_kernel<VPR>, grid, dim3(kCompactThreads), 0, stream, a);
  return hipGetLastError();
}

}  // namespace

hipError_t launch_compact(const CompactLaunch& a, hipStream_t stream) {
  if (a.C == 0) return hipSuccess;
  switch (a.row_vecs) {  // D in {64, 128} x element size in {2, 4}
    case 8: return launch_compact_t<8>(a, stream);
    case 16: return launch_compact_t<16>(a, stream);
    case 32: return launch_compact_t<32>(a, stream);
    default: return hipErrorInvalidValue;
  }
}

hipError_t launch_compact_slots(const CompactLaunch& a, hipStream_t stream) {
  if (a.C == 0) return hipSuccess;
  if (!a.slots || a.k_out != a.k || a.v_out != a.v) return hipErrorInvalidValue;
  switch (a.row_vecs) {
    case 8: hipLaunchKernelGGL(compact_slots_kernel<8>, dim3(a.B * a.H), dim3(kSlotThreads), 0, stream, a); break;
    case 16: hipLaunchKernelGGL(compact_slots_kernel<16>, dim3(a.B * a.H), dim3(kSlotThreads), 0, stream, a); break;
    case 32: hipLaunchKernelGGL(compact_slots_kernel<32>, dim3(a.B * a.H), dim3(kSlotThreads), 0, stream, a); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

hipError_t launch_append(const AppendLaunch& a, hipStream_t stream) {
  if (a.m == 0) return hipSuccess;
  if (a.row_vecs <= 0 || kCompactThreads % a.row_vecs != 0) return hipErrorInvalidValue;
  const int rows_per_block = kCompactThreads / a.row_vecs;
  dim3 grid((a.m + rows_per_block - 1) / rows_per_block, a.B * a.H, 2);
  hipLaunchKernelGGL(append_kernel, grid, dim3(kCompactThreads), 0, stream, a);
  return hipGetLastError();
}

}  // namespace nacl
