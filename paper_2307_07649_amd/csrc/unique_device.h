// Device-side pieces of the counting sort of slots by node row (see k_unique.hip).  The scan and the fill
// are small, so they do not get launches of their own in the training step: the scan (one block) rides in the node
// launch, the fill in the attention launch.
#pragma once
#include "tgnn_internal.h"

namespace tgnn {

// Exclusive scan of the slot counts gcnt[ulist[row]], row in [0, U), into rowptr[0 .. U] and cursor[0 .. U) by one
// block (any multiple of 64 threads up to 1024); the counts are cleared on the way, for the next step.  A thread takes
// PER consecutive rows at a time, all their loads at once: the block is one workgroup beside hundreds, and on 11,000 rows
// a walk with four rows per lane was 30 dependent round trips long and outlived the launch it rides in by 12 us.
// rowptr, cursor and ulist must be 16-byte aligned.
template <int PER>
__device__ __forceinline__ void uniq_scan_rows(const SortArgs& a, int U, int* wsum) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, waves = blockDim.x >> 6;
  int base = 0;
  for (int i0 = 0; i0 < U; i0 += (int)blockDim.x * PER) {
    const int i = i0 + (int)threadIdx.x * PER;
    int id[PER], v[PER], t = 0;
#pragma unroll
    for (int u = 0; u < PER; u += 4) {
      int4 q = make_int4(0, 0, 0, 0);
      if (i + u < U) q = *reinterpret_cast<const int4*>(a.ulist + i + u);   // (the list is padded to whole int4s)
      id[u] = q.x; id[u + 1] = q.y; id[u + 2] = q.z; id[u + 3] = q.w;
    }
#pragma unroll
    for (int u = 0; u < PER; ++u) v[u] = i + u < U ? a.gcnt[id[u]] : 0;
#pragma unroll
    for (int u = 0; u < PER; ++u) {
      if (i + u < U) a.gcnt[id[u]] = 0;
      t += v[u];
    }
    int inc = t;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
      const int o = __shfl_up(inc, off);
      if (lane >= off) inc += o;
    }
    __syncthreads();   // (the round before has been read)
    if (lane == 63) wsum[wave] = inc;
    __syncthreads();
    int e = base + inc - t;
    for (int w = 0; w < waves; ++w) {
      if (w < wave) e += wsum[w];
      base += wsum[w];
    }
#pragma unroll
    for (int u = 0; u < PER; u += 4) {
      const int4 q = make_int4(e, e + v[u], e + v[u] + v[u + 1], e + v[u] + v[u + 1] + v[u + 2]);
      e = q.w + v[u + 3];
      if (i + u + 3 < U) {
        *reinterpret_cast<int4*>(a.rowptr + i + u) = q;
        *reinterpret_cast<int4*>(a.cursor + i + u) = q;
      } else {
        const int r[4] = {q.x, q.y, q.z, q.w};
        for (int k = 0; k < 4; ++k)
          if (i + u + k < U) { a.rowptr[i + u + k] = r[k]; a.cursor[i + u + k] = r[k]; }
      }
    }
  }
  if (threadIdx.x == 0) {
    a.rowptr[U] = base;
    *a.total = base;
  }
}
__device__ __forceinline__ void uniq_scan_block(const SortArgs& a) {
  __shared__ int wsum[16];
  const int U = *a.ucount;
  if (U <= 4 * (int)blockDim.x) uniq_scan_rows<4>(a, U, wsum);
  else uniq_scan_rows<32>(a, U, wsum);
}

// The first launch of a step and the fill pass count slots per node.  On power-law graphs one node holds a tenth of a step's slots,
// and atomics on one address complete one at a time in the L2 (tens of nanoseconds each), so the counts are first
// taken per block in an LDS table (open addressing; LDS atomics on one word cost a few cycles) and only one global
// atomic per block and distinct row follows.  A block of 256 threads takes UNIQ_PER_BLOCK consecutive slots.
constexpr int UNIQ_PER_BLOCK = 1024;
constexpr int UNIQ_TABLE = 2048;   // >= 2 x the distinct rows a block can meet
// (the first launch: a block of 8 wavefronts meets at most 32 roots x 16 or 8 roots x 33 distinct nodes)
constexpr int CLAIM_TABLE = 1024;
__host__ __device__ inline int uniq_blocks(int S) { return (S + UNIQ_PER_BLOCK - 1) / UNIQ_PER_BLOCK; }

template <int SIZE> struct UniqTable {
  int key[SIZE];
  int val[SIZE];
};
template <int SIZE> __device__ __forceinline__ void uniq_table_clear(UniqTable<SIZE>& t) {
  for (int i = threadIdx.x; i < SIZE; i += blockDim.x) { t.key[i] = -1; t.val[i] = 0; }
}
// the entry of `row` (inserted if absent)
template <int SIZE> __device__ __forceinline__ int uniq_table_slot(UniqTable<SIZE>& t, int row) {
  int h = (int)(((unsigned)row * 2654435761u) >> 21) & (SIZE - 1);
  for (;;) {
    const int k = atomicCAS(&t.key[h], -1, row);
    if (k == -1 || k == row) return h;
    h = (h + 1) & (SIZE - 1);
  }
}

// slot s goes to the next free position of its row's range; `block` counts the blocks that do this work
__device__ __forceinline__ void uniq_fill_block(const SortArgs& a, int block) {
  __shared__ UniqTable<UNIQ_TABLE> tab;
  uniq_table_clear(tab);
  __syncthreads();
  const int s_end = min(a.S, (block + 1) * UNIQ_PER_BLOCK);
  // the block's slots per row, then one range per row claimed from the row's cursor, then positions inside it
  int my_slot[UNIQ_PER_BLOCK / 256];
#pragma unroll
  for (int u = 0; u < UNIQ_PER_BLOCK / 256; ++u) {
    const int s = block * UNIQ_PER_BLOCK + u * 256 + (int)threadIdx.x;
    const int gid = s < s_end ? a.slot_gid[s] : -1;
    const int row = gid >= 0 ? a.uidx[gid] : -1;
    my_slot[u] = -1;
    if (row >= 0) {
      my_slot[u] = uniq_table_slot(tab, row);
      atomicAdd(&tab.val[my_slot[u]], 1);
    }
  }
  __syncthreads();
  for (int i = threadIdx.x; i < UNIQ_TABLE; i += blockDim.x)
    if (tab.key[i] >= 0) tab.val[i] = atomicAdd(a.cursor + tab.key[i], tab.val[i]);
  __syncthreads();
#pragma unroll
  for (int u = 0; u < UNIQ_PER_BLOCK / 256; ++u) {
    if (my_slot[u] >= 0) {
      const int s = block * UNIQ_PER_BLOCK + u * 256 + (int)threadIdx.x;
      const int pos = atomicAdd(&tab.val[my_slot[u]], 1);
      a.sorted[pos] = s;
      a.sorted_row[pos] = tab.key[my_slot[u]];
    }
  }
}

}  // namespace tgnn
