// Link-prediction decoder and binary cross-entropy (self-supervision by temporal edges with one sampled
// negative destination per event, Sec. 2.1 / 3.2.2).  logit(a, b) = w2 . ReLU(W_s z_a + W_d z_b + b1) + b2.
// The hidden layer is linear in {z_a | z_b} before its ReLU, so the two products are taken once per root
// (one MFMA GEMM, Pdec = z {W_s ; W_d}^T) and a pair only adds two rows: the source's W_s z is shared by its
// true and its negative pair.  Backward, the pair kernel leaves per root the gradient of its row of Pdec; the
// GEMM that maps it back to z applies the ReLU gate of the merge layer in its epilogue.
// Row layout of the (1 + J) n pairs of batch b (events before it: off; J negative sets): rows (1 + J) off + i are the
// true pairs (src_i, dst_i), rows (1 + J) off + (1 + g) n + i the pairs (src_i, neg_{g,i}); roots (2 + J) off +
// {0, n, 2n, ...} + i are src, dst, neg set 0, ...
#include "tgnn_internal.h"
#include "device_math.h"

namespace tgnn {

__device__ __forceinline__ int batch_of_row(const BatchSet& bs, int row, int mult) {
  int b = 0;
  while (b + 1 < bs.nb && row >= mult * bs.b[b + 1].ev_off) ++b;
  return b;
}

// One wavefront per event (both of its pairs), at most DP_BLOCKS blocks of four wavefronts which stride over
// the events (every block ends with one atomic per column of w2: more blocks would queue up there).  Per pair: hidden layer, logit,
// loss term, d(loss)/d(logit); per root: gradient of its Pdec row ({W_s part | W_d part}: a source receives
// the sum of its two pairs in the first half, a destination its pair in the second half, the other halves
// are zero); per block: partial sums of the w2 / b2 gradients and of the loss.
// loss = mean over batches of (1 / 2n_b) sum softplus(-+logit).
constexpr int DP_BLOCKS = 256;
__global__ __launch_bounds__(256) void dec_pair_kernel(const BatchSet* __restrict__ bsp, int dO,
                                                       const float* __restrict__ Pdec, int ldp,
                                                       const float* __restrict__ b1, const float* __restrict__ w2,
                                                       const float* __restrict__ b2, float* __restrict__ logits,
                                                       float* __restrict__ out_loss, float* __restrict__ h1, int ldh,
                                                       float* __restrict__ dPdec, float* __restrict__ g_w2,
                                                       float* __restrict__ g_b2) {
  __shared__ float red[4][260];
  const BatchSet& bs = *bsp;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  float gw[4] = {0.f, 0.f, 0.f, 0.f};  // columns lane, lane+64, lane+128, lane+192
  float gb = 0.f, lsum = 0.f;
  float bb[4], ww[4];
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const int c = lane + 64 * q;
    bb[q] = c < dO ? b1[c] : 0.f;
    ww[q] = c < dO ? w2[c] : 0.f;
  }
  const float b2v = b2[0];
  const int nneg = bs.nneg;
  for (int ev = blockIdx.x * 4 + wave; ev < bs.total; ev += gridDim.x * 4) {
    const int b = batch_of_row(bs, ev, 1);
    const int off = bs.b[b].ev_off, n = bs.b[b].n;
    const int i = ev - off;
    const size_t ra = (size_t)((2 + nneg) * off + i) * ldp;   // the source's row; the partner of pair g is n (1 + g) rows on
    const float inv = 1.0f / (2.0f * (float)n);
    float ps[4], dsrc[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int c = lane + 64 * q;
      ps[q] = c < dO ? Pdec[ra + c] + bb[q] : 0.f;
    }
    float lterm = 0.f;
    // pair 0 is the true pair (src, dst); pair 1 + g pairs the source with the negative destination of set g.  With
    // nneg sets the step stands for nneg trainers that share the positive batch (Sec. 3.2.2): the loss is the mean of
    // their losses, the gradient that of their sum, so the true pair counts nneg times in the gradient.
    for (int pr = 0; pr <= nneg; ++pr) {
      const size_t rb = ra + (size_t)(1 + pr) * n * ldp;
      float h[4], acc = 0.f;
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int c = lane + 64 * q;
        h[q] = c < dO ? fmaxf(ps[q] + Pdec[rb + dO + c], 0.f) : 0.f;
        acc += h[q] * ww[q];
      }
#pragma unroll
      for (int o = 32; o > 0; o >>= 1) acc += __shfl_xor(acc, o);
      const float lg = acc + b2v;
      const float sgm = 1.0f / (1.0f + expf(-lg));
      float dl, sp;
      if (pr == 0) {   // softplus(-logit)
        sp = fmaxf(-lg, 0.f) + log1pf(expf(-fabsf(lg)));
        dl = (sgm - 1.0f) * inv * (float)nneg;
      } else {         // softplus(logit), averaged over the sets in the loss
        sp = (fmaxf(lg, 0.f) + log1pf(expf(-fabsf(lg)))) / (float)nneg;
        dl = sgm * inv;
      }
      const int row = (1 + nneg) * off + pr * n + i;
      if (lane == 0) {
        logits[row] = lg;
        gb += dl;
      }
      lterm += sp;
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int c = lane + 64 * q;
        if (c < dO) {
          const float dh = h[q] > 0.f ? dl * ww[q] : 0.f;
          h1[(size_t)row * ldh + c] = h[q];
          dPdec[rb + c] = 0.f;
          dPdec[rb + dO + c] = dh;
          dsrc[q] += dh;
          gw[q] += dl * h[q];
        }
      }
    }
    if (lane == 0) lsum += lterm * inv / (float)bs.nb;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int c = lane + 64 * q;
      if (c < dO) {
        dPdec[ra + c] = dsrc[q];
        dPdec[ra + dO + c] = 0.f;
      }
    }
  }
#pragma unroll
  for (int q = 0; q < 4; ++q) red[wave][lane + 64 * q] = gw[q];
  if (lane == 0) { red[wave][256] = gb; red[wave][257] = lsum; }
  __syncthreads();
  if (wave == 0) {
    for (int c = lane; c < dO; c += 64) atomicAdd(g_w2 + c, red[0][c] + red[1][c] + red[2][c] + red[3][c]);
    if (lane == 0) {
      atomicAdd(g_b2, red[0][256] + red[1][256] + red[2][256] + red[3][256]);
      if (out_loss != nullptr) atomicAdd(out_loss, red[0][257] + red[1][257] + red[2][257] + red[3][257]);
    }
  }
}

void decoder_pairs(const Dims& d, const BatchSet* bs, int total, const float* Pdec, int ldp, const float* b1,
                   const float* w2, const float* b2, float* logits, float* out_loss, float* h1, float* dPdec,
                   float* g_w2, float* g_b2, hipStream_t s) {
  if (total <= 0) return;
  hipLaunchKernelGGL(dec_pair_kernel, dim3(std::min((total + 3) / 4, DP_BLOCKS)), dim3(256), 0, s, bs, d.dO, Pdec, ldp, b1,
                     w2, b2, logits, out_loss, h1, d.ldh, dPdec, g_w2, g_b2);
}

// Edge-classification head (Sec. 4 "Datasets": C classes, several true per event): hidden layer
// h = ReLU(W_s z_src + W_d z_dst + b1) from the two roots' rows of Pdec, logits W2 h + b2, cross-entropy terms
// softplus(logit) - y logit, d loss / d logit = (sigmoid(logit) - y) / (n C), and the hidden layer's gradient
// W2^T dlogit gated by the ReLU.  Roots of batch b: [src | dst] from root 2 * ev_off on.  The weight
// gradients of W2 / b2 are left to the weight-gradient GEMM (dlog^T h1).
// A workgroup takes DC_E events; both products are fp32 MFMAs (16 events x 16 columns per wavefront and round) whose
// left operands stay in LDS, and the cross-entropy is evaluated once per (event, class).  4,000 events with 56 classes:
// 77 us with a wavefront per event that went through the classes one by one (all 64 lanes evaluating the same
// exponentials), 18 us this way; the launch is then bound by its phases' latencies.
constexpr int DC_E = 16;
constexpr int DC_HP = 256 + 4, DC_LP = 256 + 4;   // LDS pitches: widest hidden layer, most classes (4 mod 64 banks)
__global__ __launch_bounds__(256) void dec_class_kernel(const BatchSet* __restrict__ bsp, int dO, int C,
                                                        const float* __restrict__ Pdec, int ldp,
                                                        const float* __restrict__ b1, const float* __restrict__ w2,
                                                        const float* __restrict__ b2, float* __restrict__ logits,
                                                        float* __restrict__ out_loss, float* __restrict__ h1, int ldh,
                                                        float* __restrict__ dPdec, float* __restrict__ dlog, int ldc) {
  typedef float floatx4 __attribute__((ext_vector_type(4)));
  __shared__ __attribute__((aligned(16))) float H[DC_E * DC_HP], L[DC_E * DC_LP];
  __shared__ const float* y_s[DC_E];
  __shared__ float inv_s[DC_E], red[4];
  __shared__ int src_s[DC_E], dst_s[DC_E];
  const BatchSet& bs = *bsp;
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int li = lane & 15, lg = lane >> 4;
  const int ev0 = blockIdx.x * DC_E, n_here = min(DC_E, bs.total - ev0);
  if (tid < DC_E) {
    const int ev = ev0 + min(tid, n_here - 1), b = batch_of_row(bs, ev, 1), off = bs.b[b].ev_off, n = bs.b[b].n, i = ev - off;
    src_s[tid] = 2 * off + i;
    dst_s[tid] = 2 * off + i + n;
    y_s[tid] = bs.b[b].labels + (size_t)i * C;
    inv_s[tid] = tid < n_here ? 1.0f / ((float)n * (float)C) : 0.f;
  }
  __syncthreads();
  const int dOp = (dO + 63) & ~63, Cp = (C + 63) & ~63;   // four k slabs of either product at a time
#pragma unroll 4
  for (int idx = tid; idx < DC_E * dOp; idx += 256) {
    const int e = idx / dOp, c = idx - e * dOp;
    float h = 0.f;
    if (c < dO) {
      h = fmaxf(Pdec[(size_t)src_s[e] * ldp + c] + b1[c] + Pdec[(size_t)dst_s[e] * ldp + dO + c], 0.f);
      if (e < n_here) h1[(size_t)(ev0 + e) * ldh + c] = h;
    }
    H[e * DC_HP + c] = h;
  }
  __syncthreads();
  float lsum = 0.f;
  for (int cb = wave; cb < Cp / 16; cb += 4) {
    const int cls = cb * 16 + li;
    const float* __restrict__ wr = w2 + (size_t)min(cls, C - 1) * dO;
    floatx4 acc = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll 1
    for (int s0 = 0; s0 < dOp / 16; s0 += 4)
#pragma unroll
    for (int s = s0; s < s0 + 4; ++s) {
      const floatx4 a4 = *reinterpret_cast<const floatx4*>(&H[li * DC_HP + 16 * s + 4 * lg]);
      float w[4];
#pragma unroll
      for (int c = 0; c < 4; ++c) {   // (columns past d_o: zeros on both sides, so that an infinite weight stays where it is)
        const int k = 16 * s + 4 * lg + c;
        const float x = wr[min(k, dO - 1)];
        w[c] = k < dO ? x : 0.f;
      }
#pragma unroll
      for (int c = 0; c < 4; ++c) acc = __builtin_amdgcn_mfma_f32_16x16x4f32(a4[c], w[c], acc, 0, 0, 0);
    }
    const float bias = b2[min(cls, C - 1)];
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const int e = 4 * lg + v;
      const float lgt = acc[v] + bias, yv = y_s[e][min(cls, C - 1)];
      const float sgm = 1.0f / (1.0f + expf(-lgt));
      const bool live = cls < C && e < n_here;
      const float dl = live ? (sgm - yv) * inv_s[e] : 0.f;
      if (live) {
        lsum += (fmaxf(lgt, 0.f) + log1pf(expf(-fabsf(lgt))) - yv * lgt) * inv_s[e];
        logits[(size_t)(ev0 + e) * C + cls] = lgt;
        dlog[(size_t)(ev0 + e) * ldc + cls] = dl;
      }
      L[e * DC_LP + cls] = dl;
    }
  }
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) lsum += __shfl_xor(lsum, o);
  if (lane == 0) red[wave] = lsum;
  __syncthreads();
  if (tid == 0 && out_loss != nullptr) atomicAdd(out_loss, (red[0] + red[1] + red[2] + red[3]) / (float)bs.nb);
  for (int cb = wave; cb * 16 < dO; cb += 4) {
    const int col = cb * 16 + li, colc = min(col, dO - 1);
    floatx4 acc = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll 1
    for (int s0 = 0; s0 < Cp / 16; s0 += 4)
#pragma unroll
    for (int s = s0; s < s0 + 4; ++s) {
      const floatx4 a4 = *reinterpret_cast<const floatx4*>(&L[li * DC_LP + 16 * s + 4 * lg]);
      float w[4];
#pragma unroll
      for (int c = 0; c < 4; ++c) {   // (classes past C likewise)
        const int k = 16 * s + 4 * lg + c;
        const float x = w2[(size_t)min(k, C - 1) * dO + colc];
        w[c] = k < C ? x : 0.f;
      }
#pragma unroll
      for (int c = 0; c < 4; ++c) acc = __builtin_amdgcn_mfma_f32_16x16x4f32(a4[c], w[c], acc, 0, 0, 0);
    }
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const int e = 4 * lg + v;
      if (col < dO && e < n_here) {
        const float gq = H[e * DC_HP + col] > 0.f ? acc[v] : 0.f;
        const size_t ra = (size_t)src_s[e] * ldp, rb = (size_t)dst_s[e] * ldp;
        dPdec[ra + col] = gq; dPdec[ra + dO + col] = 0.f;
        dPdec[rb + col] = 0.f; dPdec[rb + dO + col] = gq;
      }
    }
  }
}

// Logits of the classification head in an evaluation pass: a wavefront per event, the classes one after the other.  A
// pass returns counts decided by the sign of a logit, so its sums keep the order they have always been taken in
// (a lane's columns, then the exchange over the wavefront), not the one of the MFMAs above.
__global__ __launch_bounds__(256) void class_scores_kernel(const BatchSet* __restrict__ bsp, int dO, int C,
                                                           const float* __restrict__ Pdec, int ldp,
                                                           const float* __restrict__ b1, const float* __restrict__ w2,
                                                           const float* __restrict__ b2, float* __restrict__ logits) {
  const BatchSet& bs = *bsp;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  float bb[4];
#pragma unroll
  for (int q = 0; q < 4; ++q) bb[q] = lane + 64 * q < dO ? b1[lane + 64 * q] : 0.f;
  for (int ev = blockIdx.x * 4 + wave; ev < bs.total; ev += gridDim.x * 4) {
    const int b = batch_of_row(bs, ev, 1);
    const int off = bs.b[b].ev_off, n = bs.b[b].n;
    const size_t ra = (size_t)(2 * off + ev - off) * ldp, rb = ra + (size_t)n * ldp;   // the source's and the destination's row
    float h[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int c = lane + 64 * q;
      h[q] = c < dO ? fmaxf(Pdec[ra + c] + bb[q] + Pdec[rb + dO + c], 0.f) : 0.f;
    }
    for (int cls = 0; cls < C; ++cls) {
      const float* __restrict__ wr = w2 + (size_t)cls * dO;
      float acc = 0.f;
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int c = lane + 64 * q;
        acc += h[q] * (c < dO ? wr[c] : 0.f);
      }
#pragma unroll
      for (int o = 32; o > 0; o >>= 1) acc += __shfl_xor(acc, o);
      if (lane == 0) logits[(size_t)ev * C + cls] = acc + b2[cls];
    }
  }
}

void decoder_classes(const Dims& d, const BatchSet* bs, int total, const float* Pdec, int ldp, const float* b1,
                     const float* w2, const float* b2, float* logits, float* out_loss, float* h1, float* dPdec,
                     float* dlog, hipStream_t s) {
  if (total <= 0) return;
  hipLaunchKernelGGL(dec_class_kernel, dim3((total + DC_E - 1) / DC_E), dim3(256), 0, s, bs, d.dO, d.nC, Pdec, ldp, b1, w2, b2,
                     logits, out_loss, h1, d.ldh, dPdec, dlog, d.ldc);
}

void class_scores(const Dims& d, const BatchSet* bs, int total, const float* Pdec, int ldp, const float* b1, const float* w2,
                  const float* b2, float* logits, hipStream_t s) {
  if (total <= 0) return;
  hipLaunchKernelGGL(class_scores_kernel, dim3(std::min((total + 3) / 4, 4 * DP_BLOCKS)), dim3(256), 0, s, bs, d.dO, d.nC, Pdec,
                     ldp, b1, w2, b2, logits);
}

// An evaluation pass: the scores of an event's 1 + J pairs (pair layout of the epoch-parallel step), and the rank of its
// true pair among them.  `per` wavefronts (1 or 4) share an event, each takes every per-th pair, RK_U pairs' rows in
// flight at a time; the scores meet in LDS and one wavefront counts, a lane per negative destination.  The sum of a score
// is taken as in dec_pair_kernel (a lane's columns, then the exchange over the wavefront).  600 events with 49 negatives:
// 67 us in dec_pair_kernel (which also wrote the backward pass's rows) and 14 us for the ranks (a thread per event), now
// 8.4 us together (14.8 with an atomic per event on the sum of the reciprocal ranks).
constexpr int RK_U = 7;   // pairs per round, 28 loads in flight: the 12 or 13 pairs that four wavefronts have each of 49 negatives (the
                          // usual number) are two rounds; a round that is not full repeats the last pair
__global__ __launch_bounds__(256) void pair_rank_kernel(const BatchSet* __restrict__ bsp, int dO, const float* __restrict__ Pdec,
                                                        int ldp, const float* __restrict__ b1, const float* __restrict__ w2,
                                                        const float* __restrict__ b2, float* __restrict__ logits,
                                                        float* __restrict__ rank, int per) {
  __shared__ float sc[4][TGNN_MAX_NEG_SETS + 1];
  const BatchSet& bs = *bsp;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  const int sub = per == 1 ? wave : 0, part = per == 1 ? 0 : wave;
  const int ev = per == 1 ? blockIdx.x * 4 + wave : blockIdx.x;
  const bool mine = ev < bs.total;
  const int b = mine ? batch_of_row(bs, ev, 1) : 0;
  const int off = bs.b[b].ev_off, n = bs.b[b].n, J = bs.nneg;
  const size_t r0 = (size_t)(1 + J) * off + (ev - off);
  if (mine) {
    float bb[4], ww[4], ps[4];
    const size_t ra = (size_t)((2 + J) * off + ev - off) * ldp;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int c = lane + 64 * q;
      bb[q] = c < dO ? b1[c] : 0.f;
      ww[q] = c < dO ? w2[c] : 0.f;
      ps[q] = c < dO ? Pdec[ra + c] + bb[q] : 0.f;
    }
    const float b2v = b2[0];
    for (int p0 = part; p0 <= J; p0 += per * RK_U) {
      float x[RK_U][4], acc[RK_U];
#pragma unroll
      for (int i = 0; i < RK_U; ++i) {
        const size_t rb = ra + (size_t)(1 + min(p0 + i * per, J)) * n * ldp + dO;
#pragma unroll
        for (int q = 0; q < 4; ++q)
          if (64 * q < dO) x[i][q] = Pdec[rb + min(lane + 64 * q, dO - 1)];
      }
#pragma unroll
      for (int i = 0; i < RK_U; ++i) {
        acc[i] = 0.f;
#pragma unroll
        for (int q = 0; q < 4; ++q)
          if (64 * q < dO) {
            const float h = lane + 64 * q < dO ? fmaxf(ps[q] + x[i][q], 0.f) : 0.f;
            acc[i] += h * ww[q];
          }
      }
#pragma unroll
      for (int o = 32; o > 0; o >>= 1)
#pragma unroll
        for (int i = 0; i < RK_U; ++i) acc[i] += __shfl_xor(acc[i], o);
#pragma unroll
      for (int i = 0; i < RK_U; ++i)
        if (lane == 0 && p0 + i * per <= J) sc[sub][p0 + i * per] = acc[i] + b2v;
    }
  }
  __syncthreads();
  if (!mine || part != 0) return;
  const float st = sc[sub][0], sn = sc[sub][1 + min(lane, J - 1)];
  const int above = __popcll(__ballot(lane < J && sn > st)), same = __popcll(__ballot(lane < J && sn == st));
  if (lane < J) logits[r0 + (size_t)(1 + lane) * n] = sn;
  if (lane == 0) {
    logits[r0] = st;
    rank[ev] = 1.0f + (float)above + 0.5f * (float)same;   // (the reciprocals are added up in the write-back launch)
  }
}

void pair_ranks(const Dims& d, const BatchSet* bs, int total, int nneg, const float* Pdec, int ldp, const float* b1,
                const float* w2, const float* b2, float* logits, float* rank, hipStream_t s) {
  static_assert(TGNN_MAX_NEG_SETS <= 64, "a lane per negative destination");
  if (total <= 0) return;
  const int per = nneg >= 8 ? 4 : 1;   // (fewer pairs than that do not feed four wavefronts)
  hipLaunchKernelGGL(pair_rank_kernel, dim3(per == 4 ? total : (total + 3) / 4), dim3(256), 0, s, bs, d.dO, Pdec, ldp, b1, w2, b2,
                     logits, rank, per);
}

// Predictions of the classification head against the targets: one thread per (event, class), counts summed per
// block before the three device-wide atomics.
__global__ __launch_bounds__(256) void class_count_kernel(const BatchSet* __restrict__ bsp, int C,
                                                          const float* __restrict__ logits, int32_t* __restrict__ counts) {
  __shared__ int red[3];
  const BatchSet& bs = *bsp;
  if (threadIdx.x < 3) red[threadIdx.x] = 0;
  __syncthreads();
  const long long i = blockIdx.x * 256ll + threadIdx.x;
  int tp = 0, fp = 0, fn = 0;
  if (i < (long long)bs.total * C) {
    const int ev = (int)(i / C), cls = (int)(i - (long long)ev * C);
    const int b = batch_of_row(bs, ev, 1);
    const bool y = bs.b[b].labels[(size_t)(ev - bs.b[b].ev_off) * C + cls] > 0.5f;
    const bool pred = logits[i] > 0.f;
    tp = pred && y; fp = pred && !y; fn = !pred && y;
  }
  const int ntp = __popcll(__ballot(tp)), nfp = __popcll(__ballot(fp)), nfn = __popcll(__ballot(fn));
  if ((threadIdx.x & 63) == 0) {
    if (ntp) atomicAdd(&red[0], ntp);
    if (nfp) atomicAdd(&red[1], nfp);
    if (nfn) atomicAdd(&red[2], nfn);
  }
  __syncthreads();
  if (threadIdx.x < 3 && red[threadIdx.x] != 0) atomicAdd(counts + threadIdx.x, red[threadIdx.x]);
}

void class_counts(const BatchSet* bs, int total, int C, const float* logits, int32_t* counts, hipStream_t s) {
  if (total <= 0) return;
  const long long n = (long long)total * C;
  hipLaunchKernelGGL(class_count_kernel, dim3((int)((n + 255) / 256)), dim3(256), 0, s, bs, C, logits, counts);
}

__global__ void mask_dz_kernel(int R, int dO, const float* __restrict__ dz_in, int p_in, const float* __restrict__ z,
                               int ldz, float* __restrict__ dz_out) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= R * dO) return;
  const int r = i / dO, c = i - r * dO;
  dz_out[(size_t)r * ldz + c] = z[(size_t)r * ldz + c] > 0.f ? dz_in[(size_t)r * p_in + c] : 0.f;
}

void mask_dz(int R, int dO, const float* dz_in, int p_in, const float* z, int ldz, float* dz_out, hipStream_t s) {
  if (R <= 0) return;
  hipLaunchKernelGGL(mask_dz_kernel, dim3((R * dO + 255) / 256), dim3(256), 0, s, R, dO, dz_in, p_in, z, ldz, dz_out);
}

__global__ void attn_dx_out_kernel(int R, int RK, int dm, const float* __restrict__ ds_row, int ldh,
                                   float* __restrict__ d_x_root, float* __restrict__ d_x_nbr) {
  const long long i = blockIdx.x * (long long)blockDim.x + threadIdx.x;
  if (i >= (long long)(R + RK) * dm) return;
  const int row = (int)(i / dm), c = (int)(i - (long long)row * dm);
  const float x = ds_row[(size_t)row * ldh + c];
  if (row < R) d_x_root[(size_t)row * dm + c] = x;
  else d_x_nbr[(size_t)(row - R) * dm + c] = x;
}

void attn_dx_out(int R, int RK, int dm, const float* ds_row, int ldh, float* d_x_root, float* d_x_nbr, hipStream_t s) {
  const long long total = (long long)(R + RK) * dm;
  if (total <= 0) return;
  hipLaunchKernelGGL(attn_dx_out_kernel, dim3((int)((total + 255) / 256)), dim3(256), 0, s, R, RK, dm, ds_row, ldh,
                     d_x_root, d_x_nbr);
}

__global__ void zero_kernel(float* p, int n) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) p[i] = 0.f;
}
void zero_f32(float* p, int n, hipStream_t s) {
  if (n > 0) hipLaunchKernelGGL(zero_kernel, dim3((n + 255) / 256), dim3(256), 0, s, p, n);
}

}  // namespace tgnn
