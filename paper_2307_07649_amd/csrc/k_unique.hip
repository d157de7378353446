// Distinct-node bookkeeping of a step.  UPDT (Eq. 3) depends only on a node's stored state, so every slot
// that refers to the same (replica, node) gets the same s'.  The step therefore evaluates the GRU once per
// distinct node ("row") and lets slots point at rows; this is an exact shortcut of the per-reference
// re-computation of Sec. 3.2.1.  The attention projections are linear in their input, so their node part
// is taken per row as well.  The backward pass needs, per row, the sum of the gradients of its slots:
// slots are counting-sorted by row and reduced in fixed chunks, so a node referenced thousands of times
// (power-law graphs) costs a few dozen atomic row updates instead of thousands.
#include "tgnn_internal.h"
#include "unique_device.h"
#include "qphi_device.h"

namespace tgnn {

SortArgs sort_args(tgnn_ctx* ctx, int S) {
  Ws& w = ctx->w;
  SortArgs a;
  a.ucount = w.ucount; a.gcnt = w.gcnt; a.ulist = w.ulist; a.rowptr = w.rowptr; a.cursor = w.cursor;
  a.S = S; a.slot_gid = w.slot_gid; a.uidx = w.uidx; a.sorted = w.sorted;
  a.sorted_row = w.sorted_row; a.total = w.sort_total;
  return a;
}

// Per-row sums of the slot gradients that reach the per-node projections P = {K | V || q | merge}:
//   neighbour slot (r, j) : dP[row, 0 .. 2 d_o)          += {ds[r, h, j] q[r] | p[r, h, j] dO[r]}   (per head h: the
//                           gradients of the slot's key and value rows, formed here instead of being stored)
//   root slot r           : dP[row, half .. half + 2 d_o) += {dq[r] | dz[r]}          (half = the pitch of {K | V})
// One wavefront owns SEG_CHUNK consecutive entries of the row-sorted slot list and sums runs of one row in registers.  A run
// that lies within a workgroup's entries is stored; one that goes on in another workgroup's leaves as atomic updates, one per
// workgroup and half of the row.
// element c < 2 d_o of the gradient of neighbour slot `sl` (= r k + j)
__device__ __forceinline__ float slot_grad(const SlotGrads& g, int sl, int c) {
  const int r = sl / g.k, j = sl - r * g.k;
  if (c < g.dO) return g.dscore[(size_t)r * g.H * g.k + (c / g.dh) * g.k + j] * g.Qroot[(size_t)r * g.ldh + c];
  const int cc = c - g.dO;
  return g.prob[(size_t)r * g.H * g.k + (cc / g.dh) * g.k + j] * g.dOmat[(size_t)r * g.ldh + cc];
}

#ifndef TGNN_SEG_CHUNK
#define TGNN_SEG_CHUNK 16
#endif
constexpr int SEG_CHUNK = TGNN_SEG_CHUNK;
constexpr int SEG_WAVES = 4;   // wavefronts per workgroup
// What bounds it: a wavefront's two dependent round trips (slot ids, then rows), so what counts is how many wavefronts a
// SIMD holds.  With up to two heads (TWO) the score gradients and softmax weights of a whole chunk are one gather, a lane
// per (slot, head, which of the two), handed out by readlane and chosen per column, instead of four loads and registers
// per slot and column.  A run of equal rows that lies inside the chunk belongs to this wavefront alone and is stored; only
// runs that go on in a neighbouring chunk need atomics (dP is cleared by the node launches).
// Against four loads per slot and column and atomics throughout: 51.7 -> 49.1 us on 132,000 slots of 11,000 rows (102 instead
// of 150 registers); with the atomics gone from most rows, 8 replicas 698 -> 682 us a step, 4,000 events 505 -> 490.
// (Two or four chunks per wavefront, so that a popular row costs fewer atomic updates: slower on 600 and on 4,000 events.)
// On power-law graphs one row holds a good part of the list, and atomics on one address complete one at a time: the
// launch ended 5 us after its last wavefront (600 events).  A run that goes on from one wavefront of the workgroup into the next
// is therefore put together in LDS first, by the wavefront in whose chunk it begins: one atomic update of the row per
// workgroup.  Runs between a chunk's first and last one are stored from one copy of the code.  Launches: 4,000 events 48.5 -> 32.8 us,
// eight replicas 42.7 -> 34, 600 events 12.6 -> 9.5.  (Eight wavefronts per workgroup: the same on these, 8.4 instead of 7.3 us on
// 200 events; sixteen: 13.4, 40 and 42.)
template <bool TWO>
__global__ __launch_bounds__(64 * SEG_WAVES) void seg_reduce_kernel(int R, int S, int dO, const int32_t* __restrict__ sort_total,
                                                         const int32_t* __restrict__ sorted,
                                                         const int32_t* __restrict__ sorted_row,
                                                         SlotGrads sg, int ldkv, float* __restrict__ dP, int ldp,
                                                         QPhi qphi) {
  int block = blockIdx.x;
  warm_kernargs(R, S, dO, sort_total, sorted, sorted_row, sg, ldkv, dP, ldp, qphi);
  if (qphi.part != nullptr) {   // the first blocks are passengers: gradients through the query's Phi(0)
    const int nq = qphi_blocks(qphi);
    if (block < nq) {
      qphi_block(qphi, block);
      return;
    }
    block -= nq;
  }
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6)), p0 = (block * SEG_WAVES + wave) * SEG_CHUNK;
  // what a wavefront's first run leaves to the wavefront before: which halves of the row it has, 4 more if it fills the chunk
  // and goes on (-1: nothing); and its sums
  __shared__ int left_state[SEG_WAVES];
  __shared__ float left[SEG_WAVES][8][64];
  // lanes fetch the chunk's slot ids and rows in parallel, and the rows of the entries after and before it (lanes
  // SEG_CHUNK, SEG_CHUNK + 1), without waiting for the length of the list (entries past it are dropped below); they are
  // broadcast afterwards
  int my_slot = -1, my_row = -1;
  const int at = lane <= SEG_CHUNK ? p0 + lane : p0 - 1;
  if (lane < SEG_CHUNK + 2 && at >= 0 && at < S) {
    my_slot = sorted[at];
    my_row = sorted_row[at];
  }
  const int total = *sort_total;
  if (block * SEG_WAVES * SEG_CHUNK >= total) return;   // (uniform for the workgroup)
  if (at >= total) my_slot = my_row = -1;
  const int next_row = __builtin_amdgcn_readlane(my_row, SEG_CHUNK), prev_row = __builtin_amdgcn_readlane(my_row, SEG_CHUNK + 1);
  // a neighbour slot's root and position among the root's neighbours: one division per slot, done by the lane that
  // fetched it, not one per element
  int my_r = 0, my_j = 0;
  if (my_slot >= R) {
    const int sl = my_slot - R;
    my_r = sl / sg.k;
    my_j = sl - my_r * sg.k;
  }
  const int HK = sg.H * sg.k;
  static_assert(SEG_CHUNK * 4 <= 64, "a lane per slot, head and weight");
  float my_w = 1.f;
  if (TWO) {   // (one head: the second one's lanes repeat the first's)
    const int i = lane >> 2, h = min((lane >> 1) & 1, sg.H - 1);
    const int wr = __shfl(my_r, i), wj = __shfl(my_j, i), ws = __shfl(my_slot, i);
    const float* src = (lane & 1) ? sg.prob : sg.dscore;
    if (i < SEG_CHUNK && ws >= R) my_w = src[(size_t)wr * HK + h * sg.k + wj];
  }
  for (int cb = 0; cb < dO; cb += 128) {   // 128 columns of each of the two sections per pass, 2 + 2 per lane
    // this lane's columns (the same in the key / query section and in the value / merge section) and their head
    int ck[2], head[2];
    bool live[2];
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      const int c = cb + lane + 64 * u;
      live[u] = c < dO;
      ck[u] = live[u] ? c : 0;
      head[u] = ck[u] / sg.dh;
    }
    // a run's sums {K, V, Q, M} and which halves of the row it has (1: {K | V}, 2: {Q | M})
    struct Run {
      float k[2], v[2], q[2], m[2];
      int row, has;
    };
    Run cur, first;   // the run at hand; the chunk's first one, once it has ended
    auto clear = [&](Run& r, int row) __attribute__((always_inline)) {
#pragma unroll
      for (int u = 0; u < 2; ++u) r.k[u] = r.v[u] = r.q[u] = r.m[u] = 0.f;
      r.row = row; r.has = 0;
    };
    clear(cur, -1);
    clear(first, -1);
    if (cb > 0) __syncthreads();   // the pass before has been read
    auto store = [&](const Run& r) __attribute__((always_inline)) {   // a run that no other wavefront has a part of
      float* row = dP + (size_t)r.row * ldp;
#pragma unroll
      for (int u = 0; u < 2; ++u) {
        if (live[u] && (r.has & 1)) { row[ck[u]] = r.k[u]; row[dO + ck[u]] = r.v[u]; }
        if (live[u] && (r.has & 2)) { row[ldkv + ck[u]] = r.q[u]; row[ldkv + dO + ck[u]] = r.m[u]; }
      }
    };
    auto add = [&](const Run& r) __attribute__((always_inline)) {
      float* row = dP + (size_t)r.row * ldp;
#pragma unroll
      for (int u = 0; u < 2; ++u) {
        if (live[u] && (r.has & 1)) { atomicAdd(row + ck[u], r.k[u]); atomicAdd(row + dO + ck[u], r.v[u]); }
        if (live[u] && (r.has & 2)) { atomicAdd(row + ldkv + ck[u], r.q[u]); atomicAdd(row + ldkv + dO + ck[u], r.m[u]); }
      }
    };
    int slots[SEG_CHUNK], rows[SEG_CHUNK];
#pragma unroll
    for (int i = 0; i < SEG_CHUNK; ++i) {
      // (readlane: the values are the same for every lane, so they live in scalar registers)
      slots[i] = __builtin_amdgcn_readlane(my_slot, i);
      rows[i] = __builtin_amdgcn_readlane(my_row, i);
    }
    // all row loads of the chunk are issued before any is consumed.  Which arrays a slot reads is uniform over the
    // wavefront (a root slot: its dq and dz rows; a neighbour slot: its root's q and dO rows with the slot's score
    // gradient and softmax weight per head: dK = ds q, dV = p dO)
    float xa[SEG_CHUNK][2], xb[SEG_CHUNK][2], wa[TWO ? 1 : SEG_CHUNK][2], wb[TWO ? 1 : SEG_CHUNK][2];
#pragma unroll
    for (int i = 0; i < SEG_CHUNK; ++i) {
      const bool on = rows[i] >= 0;
      const bool root = slots[i] < R;
      const int rr = __builtin_amdgcn_readlane(my_r, i);
      const size_t ro = (size_t)(root ? max(slots[i], 0) : rr);
      const float* pa = (root ? sg.dq : sg.Qroot) + ro * sg.ldh;
      const float* pb = (root ? sg.dz : sg.dOmat) + ro * sg.ldh;
#pragma unroll
      for (int u = 0; u < 2; ++u) {
        const bool ld = on && live[u];
        xa[i][u] = ld ? pa[ck[u]] : 0.f;
        xb[i][u] = ld ? pb[ck[u]] : 0.f;
        if (!TWO) {
          const size_t wo = ro * HK + __builtin_amdgcn_readlane(my_j, i) + head[u] * sg.k;
          wa[i][u] = (ld && !root) ? sg.dscore[wo] : 1.f;
          wb[i][u] = (ld && !root) ? sg.prob[wo] : 1.f;
        }
      }
    }
#pragma unroll
    for (int i = 0; i < SEG_CHUNK; ++i) {
      if (i > 0 && rows[i] != rows[i - 1]) {   // (uniform.  An entry past the list has row -1: nothing is stored for it)
        if (cur.row == rows[0] && first.row < 0) first = cur;
        else if (cur.row >= 0) store(cur);
        clear(cur, -1);
      }
      cur.row = rows[i];
      if (rows[i] >= 0) {
        if (slots[i] < R) {
          cur.has |= 2;
#pragma unroll
          for (int u = 0; u < 2; ++u) { cur.q[u] += xa[i][u]; cur.m[u] += xb[i][u]; }
        } else {
          cur.has |= 1;
          float w[4];
          if (TWO) {
#pragma unroll
            for (int q = 0; q < 4; ++q)
              w[q] = __uint_as_float(__builtin_amdgcn_readlane(__float_as_uint(my_w), 4 * i + q));
          }
#pragma unroll
          for (int u = 0; u < 2; ++u) {
            cur.k[u] += xa[i][u] * (TWO ? (head[u] > 0 ? w[2] : w[0]) : wa[TWO ? 0 : i][u]);
            cur.v[u] += xb[i][u] * (TWO ? (head[u] > 0 ? w[3] : w[1]) : wb[TWO ? 0 : i][u]);
          }
        }
      }
    }
    const bool goes_on = cur.row >= 0 && next_row == cur.row;   // the last run, in the next chunk
    const bool one = cur.row == rows[0];                        // the chunk is one run
    if (one) first = cur;
    const bool began = first.row >= 0 && prev_row == first.row;   // the first run, in the chunk before
    int left_here = -1;
    if (began && wave > 0) {   // ... by the wavefront before, which puts the run together
#pragma unroll
      for (int u = 0; u < 2; ++u) {
        left[wave][u][lane] = first.k[u]; left[wave][2 + u][lane] = first.v[u];
        left[wave][4 + u][lane] = first.q[u]; left[wave][6 + u][lane] = first.m[u];
      }
      left_here = first.has + (one && goes_on ? 4 : 0);
    } else if (!one && first.row >= 0) {
      if (began) add(first);
      else store(first);
    }
    if (lane == 0) left_state[wave] = left_here;
    __syncthreads();
    if (cur.row >= 0 && !(one && began && wave > 0)) {
      bool ends = !goes_on;
#pragma unroll 1
      for (int w = wave + 1; w < SEG_WAVES && !ends; ++w) {
        const int state = left_state[w];
#pragma unroll
        for (int u = 0; u < 2; ++u) {
          cur.k[u] += left[w][u][lane]; cur.v[u] += left[w][2 + u][lane]; cur.q[u] += left[w][4 + u][lane]; cur.m[u] += left[w][6 + u][lane];
        }
        cur.has |= state & 3;
        ends = (state & 4) == 0;
      }
      if (ends && !(one && began)) store(cur);
      else add(cur);
    }
  }
}

static SlotGrads slot_grads(tgnn_ctx* ctx, int R) {
  const Dims& d = ctx->d;
  Ws& w = ctx->w;
  SlotGrads g;
  g.dscore = w.dscore; g.prob = w.prob; g.Qroot = w.Qroot; g.dOmat = w.dOmat; g.dq = w.dq; g.dz = w.dz;
  g.R = R; g.k = d.k; g.H = d.H; g.dO = d.dO; g.dh = d.dO / d.H; g.ldh = d.ldh;
  return g;
}

void seg_reduce(tgnn_ctx* ctx, int R, int S, const QPhi& qphi, hipStream_t s) {
  const Dims& d = ctx->d;
  Ws& w = ctx->w;
  const int waves = (S + SEG_CHUNK - 1) / SEG_CHUNK;
  const dim3 grid((waves + SEG_WAVES - 1) / SEG_WAVES + qphi_blocks(qphi));
#define TGNN_SEG_CASE(TWO)                                                                                             \
  hipLaunchKernelGGL(seg_reduce_kernel<TWO>, grid, dim3(64 * SEG_WAVES), 0, s, R, S, d.dO, w.sort_total, w.sorted, w.sorted_row,  \
                     slot_grads(ctx, R), d.ldkv, w.dP, d.ldp, qphi)
  if (d.H <= 2) TGNN_SEG_CASE(true);
  else TGNN_SEG_CASE(false);
#undef TGNN_SEG_CASE
}

// slot = row: dP[r] = {0 || dq[r] | dz[r]} for roots, dP[R + j] = {dKV[j] || 0} for neighbour slots
__global__ __launch_bounds__(256) void slots_to_dp_kernel(int R, int RK, int dO, SlotGrads sg, int ldkv,
                                                          float* __restrict__ dP, int ldp, QPhi qphi) {
  int block = blockIdx.x;
  if (qphi.part != nullptr) {   // the first blocks are passengers: gradients through the query's Phi(0)
    const int nq = qphi_blocks(qphi);
    if (block < nq) {
      qphi_block(qphi, block);
      return;
    }
    block -= nq;
  }
  const long long i = block * (long long)blockDim.x + threadIdx.x;
  if (i >= (long long)(R + RK) * ldp) return;
  const int row = (int)(i / ldp), c = (int)(i - (long long)row * ldp);
  float x = 0.f;
  if (row < R) {
    const int cc = c - ldkv;
    if (cc >= 0 && cc < dO) x = sg.dq[(size_t)row * sg.ldh + cc];
    else if (cc >= dO && cc < 2 * dO) x = sg.dz[(size_t)row * sg.ldh + (cc - dO)];
  } else if (c < 2 * dO) {
    x = slot_grad(sg, row - R, c);
  }
  dP[i] = x;
}

void slots_to_dp(tgnn_ctx* ctx, int R, int RK, const QPhi& qphi, hipStream_t s) {
  const Dims& d = ctx->d;
  Ws& w = ctx->w;
  const long long total = (long long)(R + RK) * d.ldp;
  if (total <= 0) return;
  hipLaunchKernelGGL(slots_to_dp_kernel, dim3((int)((total + 255) / 256) + qphi_blocks(qphi)), dim3(256), 0, s, R, RK, d.dO,
                     slot_grads(ctx, R), d.ldkv, w.dP, d.ldp, qphi);
}

// debug: per-slot view of per-row data
__global__ void expand_rows_kernel(int S, int dm, const int32_t* __restrict__ slot_row, const float* __restrict__ src,
                                   int ld, const double* __restrict__ src_d, float* __restrict__ dst,
                                   double* __restrict__ dst_d) {
  const long long i = blockIdx.x * (long long)blockDim.x + threadIdx.x;
  if (dst != nullptr) {
    if (i >= (long long)S * dm) return;
    const int s = (int)(i / dm), c = (int)(i - (long long)s * dm);
    const int row = slot_row[s];
    dst[i] = row >= 0 ? src[(size_t)row * ld + c] : 0.f;
  } else {
    if (i >= S) return;
    const int row = slot_row[i];
    dst_d[i] = row >= 0 ? src_d[row] : 0.0;
  }
}

void expand_rows(tgnn_ctx* ctx, int S, const float* src, int ld, const double* src_d, float* dst, double* dst_d,
                 hipStream_t s) {
  const long long total = dst ? (long long)S * ctx->d.dm : S;
  if (total <= 0) return;
  hipLaunchKernelGGL(expand_rows_kernel, dim3((int)((total + 255) / 256)), dim3(256), 0, s, S, ctx->d.dm,
                     ctx->w.slot_row, src, ld, src_d, dst, dst_d);
}

}  // namespace tgnn
