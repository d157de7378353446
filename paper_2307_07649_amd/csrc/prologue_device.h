// Device side of the prologue (weight packing, clears, descriptor copies; see PrologueArgs), callable from any
// kernel: the work is laid out on a grid of nbx x prologue_rows() blocks of any size; (bx, y) is the
// calling block's place in it.
#pragma once
#include "tgnn_internal.h"
#include "device_math.h"
#include "split3.h"

namespace tgnn {

// where element (row n, column k) of a split operand with ks slabs and `groups` interleaved operands lives (part 0)
__device__ __forceinline__ size_t split_place(int n, int k, int ks, int groups, int group) {
  return ((size_t)((n >> 4) * ks + (k >> 5)) * groups + group) * 1536 + (((k & 31) >> 3) * 16 + (n & 15)) * 8 + (k & 7);
}

// The composite weights of the score vectors (see PrologueArgs::Wu_s), on nbx * PRO_COMP blocks.  A wavefront takes 64
// consecutive columns c of one head (its loads of W_k are coalesced) and four columns j of x.  The head's rows of W_k come
// in runs of 25, all loads of a run at once: a whole number of runs for the widths in most use (heads of 25, 50 and 100), and few
// enough registers for the sampler's blocks of the same launch; other widths repeat the head's last row up to the end of a
// run (heads of 32: 18 idle loads in 50, of 64: 11 in 75).
constexpr int PRO_COMP = 4;   // grid rows
__device__ __forceinline__ void prologue_composite(const PrologueArgs& a, int block, int blocks) {
  const int lane = threadIdx.x & 63, wpb = blockDim.x >> 6;
  const int dh = a.dO / a.H, c_chunks = (a.dc + 63) >> 6;
  constexpr int JW = 4;
  const int j_chunks = (a.dx + JW - 1) / JW, hc_all = a.H * c_chunks, total = hc_all * j_chunks;
  for (int i = __builtin_amdgcn_readfirstlane(block + blocks * (int)(threadIdx.x >> 6)); i < total; i += blocks * wpb) {
    const int jc = i / hc_all, hc = i % hc_all, cc = hc % c_chunks, h = hc / c_chunks;
    const int c = min(cc * 64 + lane, a.dc - 1), n = h * a.dcp + c;
    const float* __restrict__ pk = a.wk + (size_t)h * dh * a.dkv + a.dx + c;
    const float* __restrict__ pq = a.wq + (size_t)h * dh * a.dq;
    const bool live = cc * 64 + lane < a.dc;
    float acc[JW] = {0.f, 0.f, 0.f, 0.f};
    for (int d0 = 0; d0 < dh; d0 += 64) {   // a lane brings W_q's elements of one d, broadcast below
      float q[JW];
#pragma unroll
      for (int u = 0; u < JW; ++u) q[u] = pq[(size_t)min(d0 + lane, dh - 1) * a.dq + min(jc * JW + u, a.dq - 1)];   // (past column d_x: not stored)
#pragma unroll 1
      for (int d1 = 0; d1 < min(64, dh - d0); d1 += 25) {
        float v[25];
#pragma unroll
        for (int d = 0; d < 25; ++d) v[d] = pk[(size_t)min(d0 + d1 + d, dh - 1) * a.dkv];
#pragma unroll
        for (int d = 0; d < 25; ++d)
          if (d1 + d < min(64, dh - d0)) {
#pragma unroll
            for (int u = 0; u < JW; ++u) acc[u] += v[d] * __uint_as_float(__builtin_amdgcn_readlane(__float_as_uint(q[u]), d1 + d));
          }
      }
    }
    if (live) {
#pragma unroll
      for (int u = 0; u < JW; ++u) {
        const int j = jc * JW + u;
        if (j < a.dx) {
          unsigned q[3];
          split_pair(acc[u], 0.f, q[0], q[1], q[2]);
          unsigned short* o = a.Wu_s + split_place(n, j, a.kp, 1, 0);
#pragma unroll
          for (int p = 0; p < 3; ++p) o[p * 512] = (unsigned short)q[p];
        }
      }
    }
  }
}

// rows of the block grid
__host__ __device__ inline int prologue_rows(const PrologueArgs& a) { return a.n_pack + a.zero.cnt + 1 + (a.Wu_s != nullptr ? PRO_COMP : 0); }

__device__ __forceinline__ void prologue_block(const PrologueArgs& a, int bx, int nbx, int y) {
  if (a.Wu_s != nullptr) {   // first: the longest chain of loads
    if (y < PRO_COMP) {
      prologue_composite(a, y * nbx + bx, PRO_COMP * nbx);
      return;
    }
    y -= PRO_COMP;
  }
  if (y < a.n_pack) {
    const PackDesc d = a.d[y];
    if (d.mfma_ks > 0 && d.nblk > 0) {   // MFMA B-operand order, block-diagonal
      const int per = d.rows * d.cols, total = d.nblk * per;
      for (int i = bx * blockDim.x + threadIdx.x; i < total; i += nbx * blockDim.x) {
        const int h = i / per, rc = i - h * per;
        int r, c;   // (consecutive threads walk whichever index is contiguous in the source)
        if (d.srs == 1) { c = rc / d.rows; r = rc - c * d.rows; }
        else { r = rc / d.cols; c = rc - r * d.cols; }
        const int row = h * d.brd + r, k = h * d.bcd + c;
        d.dst[((size_t)((row >> 4) * d.mfma_ks + (k >> 4)) * 64 + ((k & 15) >> 2) * 16 + (row & 15)) * 4 + (k & 3)] =
            d.src[(size_t)h * d.bsrc + (size_t)r * d.srs + (size_t)c * d.scs];
      }
      return;
    }
    if (d.mfma_ks > 0) {   // MFMA B-operand order
      const int total = ((d.rows + 15) >> 4) * d.mfma_ks * 256;
      for (int i = bx * blockDim.x + threadIdx.x; i < total; i += nbx * blockDim.x) {
        const int slab = i >> 8, t = i & 255, lane = t >> 2, c = t & 3;
        const int cb = slab / d.mfma_ks, s = slab - cb * d.mfma_ks;
        const int row = cb * 16 + (lane & 15), k = s * 16 + (lane >> 4) * 4 + c;
        d.dst[i] = (row < d.rows && k < d.cols) ? d.src[(size_t)row * d.srs + (size_t)k * d.scs] : 0.f;
      }
      return;
    }
    if (d.split_ks > 0) {   // the three bf16 parts in MFMA operand order
      unsigned short* dst = reinterpret_cast<unsigned short*>(d.dst);
      {   // eight columns per thread (col0 is a multiple of eight)
        const int c8 = (d.cols + 7) >> 3, total = d.rows * c8;
        for (int i = bx * blockDim.x + threadIdx.x; i < total; i += nbx * blockDim.x) {
          const int r = i / c8, c = (i - r * c8) * 8;
          const float* __restrict__ src = d.src + (size_t)r * d.srs + (size_t)c * d.scs;
          floatx4 lo, hi;
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            lo[e] = c + e < d.cols ? src[e * d.scs] : 0.f;
            hi[e] = c + 4 + e < d.cols ? src[(4 + e) * d.scs] : 0.f;
          }
          const Split8 s = split8(lo, hi);
          bf16x8* o = reinterpret_cast<bf16x8*>(dst + split_place(d.row0 + r, d.col0 + c, d.split_ks, d.split_groups, d.split_group));
#pragma unroll
          for (int p = 0; p < 3; ++p) o[p * 64] = s.p[p];
        }
      }
      return;
    }
    if (d.nblk > 0) {   // block-diagonal
      const int per = d.rows * d.cols, total = d.nblk * per;
      for (int i = bx * blockDim.x + threadIdx.x; i < total; i += nbx * blockDim.x) {
        const int h = i / per, rc = i - h * per;
        // consecutive threads walk whichever index is contiguous in the source
        int r, c;
        if (d.srs == 1) { c = rc / d.rows; r = rc - c * d.rows; }
        else { r = rc / d.cols; c = rc - r * d.cols; }
        d.dst[(size_t)(h * d.brd + r) * d.ldd + h * d.bcd + c] = d.src[(size_t)h * d.bsrc + (size_t)r * d.srs + (size_t)c * d.scs];
      }
      return;
    }
    const int total = d.rows * d.zero_to;
    const float* __restrict__ src = d.src;
    float* __restrict__ dst = d.dst;
    const int stride = nbx * blockDim.x;
    // four elements per pass, their loads issued together
    for (int i0 = bx * blockDim.x + threadIdx.x; i0 < total; i0 += 4 * stride) {
      float v[4];
      int off[4];
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const int i = i0 + j * stride;
        const int r = i / d.zero_to, c = i - r * d.zero_to;
        off[j] = i < total ? r * d.ldd + c : -1;
        v[j] = (i < total && c < d.cols) ? src[(size_t)r * d.srs + (size_t)c * d.scs] : 0.f;
      }
#pragma unroll
      for (int j = 0; j < 4; ++j)
        if (off[j] >= 0) dst[off[j]] = v[j];
    }
  } else if (y < a.n_pack + a.zero.cnt) {
    float* p = a.zero.p[y - a.n_pack];
    const int n = a.zero.n[y - a.n_pack];
    for (int i = bx * blockDim.x + threadIdx.x; i < n; i += nbx * blockDim.x) p[i] = 0.f;
  } else if (bx == 0) {
    if (a.bs_dev) {
      const int* src = reinterpret_cast<const int*>(&a.bs);
      int* dst = reinterpret_cast<int*>(a.bs_dev);
      for (int i = threadIdx.x; i < (int)(sizeof(BatchSet) / sizeof(int)); i += blockDim.x) dst[i] = src[i];
    }
    if (a.sgd_dev) {
      const int* src = reinterpret_cast<const int*>(&a.sgd);
      int* dst = reinterpret_cast<int*>(a.sgd_dev);
      for (int i = threadIdx.x; i < (int)(sizeof(SgdSet) / sizeof(int)); i += blockDim.x) dst[i] = src[i];
    }
    for (int i = threadIdx.x; i < a.q_part_n; i += blockDim.x) a.q_part[i] = 0.f;
    if (threadIdx.x == 0) {
      if (a.loss) *a.loss = 0.f;
      if (a.adam_t) *a.adam_t += 1;
      if (a.head_of_step) {
        *a.ucount_next = 0;
      } else {
        *a.epoch += 1ull;
        *a.ucount = 0;
      }
    }
  } else if (a.bq_out != nullptr) {
    // the query's time encoding Phi(0) = cos(time_b) does not depend on the root: fold W_q Phi(0) into the
    // bias.  One wavefront per output row, rows dealt over blocks 1 .. nbx - 1 of this grid row.
    const int lane = threadIdx.x & 63;
    const int wv = (bx - 1) * (blockDim.x >> 6) + (threadIdx.x >> 6);
    const int n_wv = (nbx - 1) * (blockDim.x >> 6);
    for (int n = wv; n < a.dO; n += n_wv) {
      float acc = 0.f;
      for (int c = lane; c < a.dt; c += 64) acc += a.wq[(size_t)n * a.dq + a.dx + c] * time_enc(0.0, 0.f, a.time_b[c]);
      for (int o = 32; o > 0; o >>= 1) acc += __shfl_xor(acc, o);
      if (lane == 0) a.bq_out[n] = a.bq[n] + acc;
    }
  }
}

}  // namespace tgnn
