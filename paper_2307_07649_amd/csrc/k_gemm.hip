// GEMMs for the dense contractions of the step: NT on fp32 MFMAs, the weight gradients (TN) on split bf16 operands.
// NT: the GRU and attention projections
// (Eq. 3-6), the merge layer, the decoder, and their data / weight gradients.
//
// v_mfma_f32_16x16x4_f32: lane l supplies A[i = l%16][kk = l/16] and B[kk = l/16][j = l%16]; its four
// accumulators hold D[i = 4*(l/16) + v][j = l%16].  The sum over kk is order independent, so a lane may
// feed any four k indices per instruction as long as both operands use the same ones: lane group g reads
// one float4 (k = 4g .. 4g+3 of a 16-wide slab) and issues four MFMAs from it.
//
// The NT kernel keeps two register tile sets in flight (global loads issued two stages ahead) and two LDS
// buffers, so a workgroup waits for memory only when the chip has nothing else resident to run.
#include <stdlib.h>

#include <algorithm>
#include <functional>
#include <cstring>

#include "tgnn_internal.h"
#include "device_math.h"
#include "split3.h"
#include "writeback_device.h"

namespace tgnn {

// A row count that an earlier kernel left in memory, read through the scalar cache (a third of the latency of a
// vector load; nothing in these kernels writes it).
__device__ __forceinline__ int load_count(const int* p) {
  return *reinterpret_cast<const int __attribute__((address_space(4)))*>(reinterpret_cast<size_t>(p));
}

// ------------------------------------------------------------------------------------------------
// NT: C = A * B^T.  One workgroup = 4 waves stacked along M (16 rows each); every wave spans the
// whole 16*TN-wide column tile.  A stage is 32 k-columns.
// ------------------------------------------------------------------------------------------------
constexpr int NT_BK = 32;
constexpr int NT_P = 32;
// LDS rows are 32 floats = 8 chunks of 16 bytes, unpadded; chunk c of row r is stored at chunk position
// c ^ ((r >> 1) & 7).  Sixteen lanes that access the same logical chunk of sixteen consecutive rows (MFMA
// operand reads), or the eight chunks of two consecutive rows (stage stores), then cover all 64 banks once.
__device__ __forceinline__ int nt_swz(int row, int chunk) { return row * NT_P + ((chunk ^ ((row >> 1) & 7)) << 2); }

// The argument block is read through the kernel-argument segment (scalar loads at a computed offset).
typedef const NtGroup __attribute__((address_space(4))) * NtGroupPtr;
// Floats of LDS that a tile of TN column blocks takes: two stage buffers of A and of B; the finished tile is staged in the same
// memory for its row-wise stores.
template <int TN> constexpr int nt_lds() { return 2 * (NT_BM + 16 * TN) * NT_P; }

// One tile of problem pi: workgroup `block` of the ones that the problem has, `col_tiles` tiles of columns, M rows.
template <int TN> __device__ __forceinline__ void nt_tile(const NtGroupPtr gp, int pi, int block, int col_tiles, int M, float* smem) {
  constexpr int BM = NT_BM, BN = 16 * TN;
  const auto& q = gp->p[pi];
  const float* __restrict__ A = q.A;
  const float* __restrict__ B = q.B;
  const float* __restrict__ bias = q.bias;
  float* __restrict__ C = q.C;
  const int lda = q.lda, ldb = q.ldb, ldc = q.ldc, N = q.N, Kp = q.Kp, n_store = q.n_store, relu = q.relu;
  RowAdd add;
  add.src = q.add.src; add.index = q.add.index; add.ld = q.add.ld; add.row0 = q.add.row0;
  add.gate = q.add.gate; add.ld_gate = q.add.ld_gate;
  TimeGradOut tg;
  tg.delta = q.tg.delta; tg.w = q.tg.w; tg.b = q.tg.b; tg.g_w = q.tg.g_w; tg.g_b = q.tg.g_b;
  GruBwdOut gb;
  gb.gates = q.gb.gates; gb.Hm = q.gb.Hm; gb.has = q.gb.has; gb.dgi = q.gb.dgi; gb.dgh = q.gb.dgh;
  gb.dm = q.gb.dm; gb.ldh = q.gb.ldh; gb.ld3 = q.gb.ld3;
  // Workgroups are dealt round-robin to the 8 XCDs, each with its own L2.  The column tiles of one row tile
  // read the same rows of A, so they are given consecutive slots of one XCD.
  const int xcd = block & 7, slot = block >> 3;
  const int row_tile = (slot / col_tiles) * 8 + xcd, col_tile = slot % col_tiles;
  if (row_tile * BM >= M) return;   // uniform for the workgroup, before any barrier
  constexpr int A_PER = BM * 8 / 256, B_F4 = BN * 8;  // float4 loads per stage and thread
  constexpr int B_PER = (B_F4 + 255) / 256;
  float (*As)[BM * NT_P] = reinterpret_cast<float (*)[BM * NT_P]>(smem);
  float (*Bs)[BN * NT_P] = reinterpret_cast<float (*)[BN * NT_P]>(smem + 2 * BM * NT_P);

  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int li = lane & 15, lg = lane >> 4;
  const int m0 = row_tile * BM, n0 = col_tile * BN;

  floatx4 acc[TN];
#pragma unroll
  for (int b = 0; b < TN; ++b) acc[b] = floatx4{0.f, 0.f, 0.f, 0.f};

  // Row indices are clamped instead of guarded, so the hot loop has no branches: rows >= M and weight
  // rows >= N read valid memory whose products are dropped in the epilogue.
  // the k range of this column tile: all of it, or with a block-diagonal B the stages its blocks reach into
  int k_lo = 0, k_hi = Kp, k_end = q.k_live > 0 ? q.k_live : Kp;
  if (q.bd_n > 0) {
    const int h_lo = min(n0, N - 1) / q.bd_n, h_hi = (min(n0 + BN, N) - 1) / q.bd_n;
    k_lo = (h_lo * q.bd_k) & ~(NT_BK - 1);
    k_end = min(k_end, (h_hi + 1) * q.bd_k);
    k_hi = min(Kp, (k_end + NT_BK - 1) & ~(NT_BK - 1));
    if (k_hi <= k_lo) k_lo = max(k_hi - NT_BK, 0);   // (live columns end before the tile's blocks begin: one stage of zeros)
  }
  const float* pa[A_PER];
  const float* pb[B_PER];
#pragma unroll
  for (int u = 0; u < A_PER; ++u) {
    const int f = tid + u * 256;
    pa[u] = A + (size_t)min(m0 + (f >> 3), M - 1) * lda + (f & 7) * 4 + k_lo;
  }
#pragma unroll
  for (int u = 0; u < B_PER; ++u) {
    const int f = min(tid + u * 256, B_F4 - 1);
    pb[u] = B + (size_t)min(n0 + (f >> 3), N - 1) * ldb + (f & 7) * 4 + k_lo;
  }
  struct Regs {
    floatx4 a[A_PER], b[B_PER];
  };
  Regs r0, r1;  // the two register tile sets
  auto gload = [&](Regs& r, int k0) __attribute__((always_inline)) {
#pragma unroll
    for (int u = 0; u < A_PER; ++u) r.a[u] = *reinterpret_cast<const floatx4*>(pa[u] + k0);
#pragma unroll
    for (int u = 0; u < B_PER; ++u) r.b[u] = *reinterpret_cast<const floatx4*>(pb[u] + k0);
  };
  auto sstore = [&](const Regs& r, int buf) __attribute__((always_inline)) {
#pragma unroll
    for (int u = 0; u < A_PER; ++u) {
      const int f = tid + u * 256;
      *reinterpret_cast<floatx4*>(&As[buf][nt_swz(f >> 3, f & 7)]) = r.a[u];
    }
#pragma unroll
    for (int u = 0; u < B_PER; ++u) {
      const int f = tid + u * 256;
      if (B_F4 % 256 == 0 || f < B_F4) *reinterpret_cast<floatx4*>(&Bs[buf][nt_swz(f >> 3, f & 7)]) = r.b[u];
    }
  };
  // the last stage stops after its first slab when the live columns end there
  const int k_tail = (q.k_live > 0 || q.bd_n > 0) ? k_end - (k_hi - NT_BK) : NT_BK;
  const bool short_tail = k_tail > 0 && k_tail <= 16;
  auto compute = [&](int buf, bool last = false) __attribute__((always_inline)) {
#pragma unroll
    for (int h = 0; h < 2; ++h) {  // two 16-wide k slabs per stage
      if (h == 1 && last && short_tail) break;
      const floatx4 a4 = *reinterpret_cast<const floatx4*>(&As[buf][nt_swz(wave * 16 + li, h * 4 + lg)]);
      floatx4 b4[TN];
#pragma unroll
      for (int b = 0; b < TN; ++b)
        b4[b] = *reinterpret_cast<const floatx4*>(&Bs[buf][nt_swz(b * 16 + li, h * 4 + lg)]);
#pragma unroll
      for (int b = 0; b < TN; ++b) acc[b] = __builtin_amdgcn_mfma_f32_16x16x4f32(a4.x, b4[b].x, acc[b], 0, 0, 0);
#pragma unroll
      for (int b = 0; b < TN; ++b) acc[b] = __builtin_amdgcn_mfma_f32_16x16x4f32(a4.y, b4[b].y, acc[b], 0, 0, 0);
#pragma unroll
      for (int b = 0; b < TN; ++b) acc[b] = __builtin_amdgcn_mfma_f32_16x16x4f32(a4.z, b4[b].z, acc[b], 0, 0, 0);
#pragma unroll
      for (int b = 0; b < TN; ++b) acc[b] = __builtin_amdgcn_mfma_f32_16x16x4f32(a4.w, b4[b].w, acc[b], 0, 0, 0);
    }
  };

  // Kp is a multiple of the stage depth.  Stage s lives in register set s & 1 until it is stored to LDS
  // buffer s & 1; loads run two stages ahead of the MFMAs.
  const int nk = (k_hi - k_lo) / NT_BK;
  // rows this lane writes: m0 + wave * 16 + lg * 4 + v.  Their gather-add source rows (or -1), and then the
  // values to add, are fetched now: two dependent loads that would otherwise sit between the last MFMA and
  // the stores.
  // The first two stages are asked for first; the index loads are four independent ones (clamped rows, no
  // branch between them: one wait, not four).
  gload(r0, 0);
  gload(r1, nk > 1 ? NT_BK : 0);
  int arow[4] = {-1, -1, -1, -1};
  if (add.src != nullptr) {
    const int row0 = m0 + wave * 16 + lg * 4;
    if (add.index != nullptr) {
      int idx[4];
#pragma unroll
      for (int v = 0; v < 4; ++v) idx[v] = add.index[min(row0 + v, M - 1)];
#pragma unroll
      for (int v = 0; v < 4; ++v) arow[v] = row0 + v < M ? idx[v] : -1;
    } else {
#pragma unroll
      for (int v = 0; v < 4; ++v) arow[v] = row0 + v < M ? row0 + v + add.row0 : -1;
    }
  }
  sstore(r0, 0);
  float addv[TN][4], bv[TN];
#pragma unroll
  for (int b = 0; b < TN; ++b) {
    const int col = n0 + b * 16 + li;
    bv[b] = (bias != nullptr && col < N) ? bias[col] : 0.f;
#pragma unroll
    for (int v = 0; v < 4; ++v)
      addv[b][v] = (add.src != nullptr && arow[v] >= 0 && col < N) ? add.src[(size_t)arow[v] * add.ld + col] : 0.f;
  }
  __syncthreads();
  int kt = 0;
  for (; kt + 3 < nk; kt += 2) {
    gload(r0, (kt + 2) * NT_BK);
    compute(0);
    sstore(r1, 1);
    __syncthreads();
    gload(r1, (kt + 3) * NT_BK);
    compute(1);
    sstore(r0, 0);
    __syncthreads();
  }
  // 1, 2 or 3 stages remain: kt (in LDS 0), kt+1 (in set 1), kt+2 (not loaded yet)
  const int rem = nk - kt;
  if (rem == 3) gload(r0, (kt + 2) * NT_BK);
  compute(0, rem == 1);
  if (rem >= 2) {
    sstore(r1, 1);
    __syncthreads();
    compute(1, rem == 2);
    if (rem == 3) {
      sstore(r0, 0);
      __syncthreads();
      compute(0, true);
    }
  }

  if (tg.g_w != nullptr) {
    // Time-encoding gradient epilogue: the tile is not stored.  Each lane multiplies its 4 rows x TN columns
    // by -sin(w_col delta_row + b_col) (the argument formed exactly as in the forward kernels), sums over its
    // rows, then over the four lane groups (shuffles) and the four waves (LDS).
    __syncthreads();   // all waves are done reading the last stage: the stage buffer becomes scratch
    float* red = &As[0][0];   // [2][4 waves][BN]
    double dl[4];
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const int row = m0 + wave * 16 + lg * 4 + v;
      dl[v] = row < M ? tg.delta[row] : 0.0;
    }
#pragma unroll
    for (int b = 0; b < TN; ++b) {
      const int col = n0 + b * 16 + li;
      float sw = 0.f, sb = 0.f;
      if (col < N) {
        const double wv = (double)tg.w[col], bv = (double)tg.b[col];
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          if (m0 + wave * 16 + lg * 4 + v < M) {
            float sn, cs;
            sincos_reduced(fma(wv, dl[v], bv), sn, cs);
            const float t = -acc[b][v] * sn;
            sb += t;
            sw += t * (float)dl[v];
          }
        }
      }
      sw += __shfl_xor(sw, 16); sw += __shfl_xor(sw, 32);
      sb += __shfl_xor(sb, 16); sb += __shfl_xor(sb, 32);
      if (lg == 0) {
        red[wave * BN + b * 16 + li] = sw;
        red[(4 + wave) * BN + b * 16 + li] = sb;
      }
    }
    __syncthreads();
    for (int c = tid; c < BN; c += 256) {
      const int col = n0 + c;
      if (col < N) {
        atomicAdd(tg.g_w + col, red[c] + red[BN + c] + red[2 * BN + c] + red[3 * BN + c]);
        atomicAdd(tg.g_b + col, red[4 * BN + c] + red[5 * BN + c] + red[6 * BN + c] + red[7 * BN + c]);
      }
    }
    return;
  }
  if (gb.dgi != nullptr) {
    // GRU gates backward epilogue: acc is the gradient reaching s' = (1 - z) n + z h.  All loads first, then
    // arithmetic and stores: a load between two stores would wait for the earlier store to complete.
    bool hs[4];
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const int row = m0 + wave * 16 + lg * 4 + v;
      hs[v] = row < M && gb.has[row] != 0;
    }
    constexpr int GB = TN < 2 ? TN : 2;   // column blocks per group (bounds the registers of wide tiles)
#pragma unroll
    for (int b0 = 0; b0 < TN; b0 += GB) {
      float gr[GB][4], gz[GB][4], gn[GB][4], ghn[GB][4], gh[GB][4];
#pragma unroll
      for (int bb = 0; bb < GB; ++bb) {
        const int col = n0 + (b0 + bb) * 16 + li;
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          const int row = m0 + wave * 16 + lg * 4 + v;
          gr[bb][v] = gz[bb][v] = gn[bb][v] = ghn[bb][v] = gh[bb][v] = 0.f;
          if (b0 + bb < TN && col < N && hs[v]) {
            const float* g = gb.gates + (size_t)row * 4 * gb.ldh;
            gr[bb][v] = g[col]; gz[bb][v] = g[gb.ldh + col]; gn[bb][v] = g[2 * gb.ldh + col];
            ghn[bb][v] = g[3 * gb.ldh + col];
            gh[bb][v] = gb.Hm[(size_t)row * gb.ldh + col];
          }
        }
      }
#pragma unroll
      for (int bb = 0; bb < GB; ++bb) {
        const int b = b0 + bb;
        const int col = n0 + b * 16 + li;
        if (b >= TN || col >= N) continue;
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          const int row = m0 + wave * 16 + lg * 4 + v;
          if (row >= M) continue;
          float drp = 0.f, dzp = 0.f, dnp = 0.f, dnr = 0.f;
          if (hs[v]) {
            const float ds = acc[b < TN ? b : 0][v];
            const float r = gr[bb][v], z = gz[bb][v], nn = gn[bb][v], hn = ghn[bb][v], h = gh[bb][v];
            const float dn = ds * (1.0f - z);
            const float dz = ds * (h - nn);
            dnp = dn * (1.0f - nn * nn);
            const float dr = dnp * hn;
            dzp = dz * z * (1.0f - z);
            drp = dr * r * (1.0f - r);
            dnr = dnp * r;
          }
          float* a = gb.dgi + (size_t)row * gb.ld3;
          float* h_ = gb.dgh + (size_t)row * gb.ld3;
          a[col] = drp; a[gb.dm + col] = dzp; a[2 * gb.dm + col] = dnp;
          h_[col] = drp; h_[gb.dm + col] = dzp; h_[2 * gb.dm + col] = dnr;
        }
      }
    }
    return;
  }
  // A lane holds 4 rows x 16-column-strided pieces of the tile: stored from here, every instruction would write
  // 64-byte pieces of four rows.  The tile goes through LDS instead and leaves as whole rows, 16 bytes per lane.
  const bool rowwise = (n_store & 3) == 0 && (ldc & 3) == 0 && (reinterpret_cast<size_t>(C) & 15) == 0;
  constexpr int CP = BN + 4;   // pitch = 4 mod 16 floats: the 4 x 16 lanes of a store hit 64 different banks
  unsigned closed = 0u;   // bit 4 b + v: the gate of that element is closed (result 0)
  if (add.gate != nullptr) {   // all gate values first: no load, and no wait for one, between the stores below
#pragma unroll
    for (int b = 0; b < TN; ++b) {
      const int col = n0 + b * 16 + li;
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const int row = m0 + wave * 16 + lg * 4 + v;
        if (col < N && row < M && !(add.gate[(size_t)row * add.ld_gate + col] > 0.f)) closed |= 1u << (4 * b + v);
      }
    }
  }
#pragma unroll
  for (int b = 0; b < TN; ++b) {
    const int col = n0 + b * 16 + li;
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const int row = m0 + wave * 16 + lg * 4 + v;
      const bool live = col < N && row < M && ((closed >> (4 * b + v)) & 1u) == 0u;
      const float x = acc[b][v] + bv[b] + addv[b][v];
      acc[b][v] = live ? (relu ? fmaxf(x, 0.f) : x) : 0.f;
    }
  }
  if (q.colsum != nullptr) {   // column sums of the tile: a lane's four rows, then the four lane groups; one atomic per wave
    float* cs = q.colsum + (size_t)((row_tile * 4 + wave) & (q.colsum_rows - 1)) * N;
#pragma unroll
    for (int b = 0; b < TN; ++b) {
      float t = acc[b][0] + acc[b][1] + acc[b][2] + acc[b][3];
      t += __shfl_xor(t, 16);
      t += __shfl_xor(t, 32);
      const int col = n0 + b * 16 + li;
      if (lg == 0 && col < N) atomicAdd(cs + col, t);
    }
  }
  if (!rowwise) {
#pragma unroll
    for (int b = 0; b < TN; ++b) {
      const int col = n0 + b * 16 + li;
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const int row = m0 + wave * 16 + lg * 4 + v;
        if (col < n_store && row < M) C[(size_t)row * ldc + col] = acc[b][v];
      }
    }
    return;
  }
  __syncthreads();   // all waves are done reading the last stage
#pragma unroll
  for (int b = 0; b < TN; ++b)
#pragma unroll
    for (int v = 0; v < 4; ++v) smem[(wave * 16 + lg * 4 + v) * CP + b * 16 + li] = acc[b][v];
  __syncthreads();
  constexpr int F4_ROW = BN / 4, F4_ALL = BM * F4_ROW;
#pragma unroll
  for (int u = 0; u < (F4_ALL + 255) / 256; ++u) {
    const int f = tid + u * 256;
    const int r = f / F4_ROW, c = (f - r * F4_ROW) * 4;
    if ((F4_ALL % 256 == 0 || f < F4_ALL) && m0 + r < M && n0 + c < n_store)
      *reinterpret_cast<floatx4*>(C + (size_t)(m0 + r) * ldc + n0 + c) = *reinterpret_cast<const floatx4*>(&smem[r * CP + c]);
  }
}

// ------------------------------------------------------------------------------------------------
// NT for few rows, the same sums in the same order.  With a tile per compute unit or less the kernel above is a chain of latencies: it
// waits for two stages of 32 columns at a time, 0.4 us each whatever the tile, thirteen of them for the widest product of a
// 600-event step.  Here a wavefront's rows of A are its own: it asks for a chunk of four stages at once and for the next one as
// it goes, and changes their order to the MFMAs' in 2 KB of LDS that no other wavefront touches (the LDS takes a
// wavefront's accesses in order), so that the only barrier is one per chunk, for the rows of B, which the four wavefronts
// share.  B is the first MFMA operand: a lane ends up with four consecutive columns of one row (column n0 + 4 lg, row m0 + 16
// wave + li), and what its epilogue needs is asked for before the last chunk, 16 bytes at a time.
// Launches of a 600-event step: 8.2, 10.3 and 8.9 -> 7.0 to 7.9 us.  Tried: operands from memory in the MFMAs' order without LDS
// (four neighbouring lanes ask for pieces of four rows, the L1 takes four times as long: 10.9 us); every wavefront its own rows of
// B (8.0); four parts of the k range on sixteen wavefronts (9.0: four times the loads of B).  With more tiles the kernel above is
// faster (see nt_tile_blocks): this one's registers leave three wavefronts per SIMD on tiles of 32 columns.
// ------------------------------------------------------------------------------------------------
constexpr int NT_CHUNK = 4;   // stages of 32 columns per chunk
constexpr int NT_FEW_TURN = 4 * 512, NT_FEW_LDS = NT_FEW_TURN + 2 * 16 * 32 * NT_CHUNK;   // floats of LDS: rows of A, two chunks of B

__device__ __forceinline__ bool aligned4(const void* p, int ld) { return ((reinterpret_cast<size_t>(p) & 15) | (ld & 3)) == 0; }
// four consecutive floats of which `live` exist (the others read as zero)
__device__ __forceinline__ floatx4 load4(const float* p, int live, bool vec) {
  floatx4 v = floatx4{0.f, 0.f, 0.f, 0.f};
  if (live >= 4 && vec) v = *reinterpret_cast<const floatx4*>(p);
  else
#pragma unroll
    for (int e = 0; e < 4; ++e)
      if (e < live) v[e] = p[e];
  return v;
}
__device__ __forceinline__ void store4(float* p, const floatx4& v, int live, bool vec) {
  if (live >= 4 && vec) *reinterpret_cast<floatx4*>(p) = v;
  else
#pragma unroll
    for (int e = 0; e < 4; ++e)
      if (e < live) p[e] = v[e];
}
// the sum over the 16 lanes of a row, in all of them
__device__ __forceinline__ float row_sum(float x) {
  x = dpp_add<0x128>(x);   // row_ror:8, 4, 2, 1
  x = dpp_add<0x124>(x);
  x = dpp_add<0x122>(x);
  return dpp_add<0x121>(x);
}

// (arguments as in nt_tile)
__device__ __forceinline__ void nt_few_tile(const NtGroupPtr gp, int pi, int block, int col_tiles, int M, float* smem) {
  constexpr int D = NT_CHUNK, KC = 32 * NT_CHUNK;
  const auto& q = gp->p[pi];
  const int N = q.N, n_store = q.n_store;
  const float* __restrict__ A = q.A;
  const float* __restrict__ B = q.B;
  const int xcd = block & 7, slot = block >> 3;
  const int row_tile = (slot / col_tiles) * 8 + xcd, col_tile = slot % col_tiles;
  if (row_tile * NT_BM >= M) return;   // uniform for the workgroup, before any barrier

  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int li = lane & 15, lg = lane >> 4;
  const int n0 = col_tile * 16, col = n0 + 4 * lg;   // this lane's columns col .. col + 3 ...
  const int row = row_tile * NT_BM + wave * 16 + li, rowc = min(row, M - 1);   // ... of this row; clamped: what comes of it is dropped
  const bool row_live = row < M;

  // the stages of 32 columns of this column tile: all of them, or with a block-diagonal B those its blocks reach into
  int k_lo = 0, k_end = q.k_live > 0 ? q.k_live : q.Kp;
  if (q.bd_n > 0) {
    const int h_lo = min(n0, N - 1) / q.bd_n, h_hi = (min(n0 + 16, N) - 1) / q.bd_n;
    k_lo = (h_lo * q.bd_k) & ~31;
    k_end = min(k_end, (h_hi + 1) * q.bd_k);
    if (k_end <= k_lo) k_lo = max(k_end - 1, 0) & ~31;   // (live columns end before the tile's blocks begin: one stage of zeros)
  }
  const int slabs = max((k_end - k_lo + 15) >> 4, 1), stages = (slabs + 1) >> 1;   // (an odd last slab: the stage's second one is left out)
  // A: eight lanes load a row's 128 bytes, a cache line; piece c of row r lies at place c ^ (r >> 1) in LDS: sixteen lanes that
  // read one piece of sixteen rows, or eight pieces of two, cover all banks
  const int lr = lane >> 3, lc = lane & 7;
  const float* pa[2];
#pragma unroll
  for (int h = 0; h < 2; ++h) pa[h] = A + (size_t)min(row_tile * NT_BM + wave * 16 + 8 * h + lr, M - 1) * q.lda + k_lo + 4 * lc;
  // B: 32 lanes load a row's 512 bytes; piece c of row r lies at place c ^ (r mod 16)
  const int br = tid >> 5, bc = tid & 31;
  const float* pb[2];
#pragma unroll
  for (int u = 0; u < 2; ++u) pb[u] = B + (size_t)min(n0 + 8 * u + br, N - 1) * q.ldb;
  float (*const Bs)[16 * KC] = reinterpret_cast<float (*)[16 * KC]>(smem + NT_FEW_TURN);
  float* const mine = smem + 512 * wave;

  floatx4 ra[D][2], rb[2], acc = floatx4{0.f, 0.f, 0.f, 0.f};
  struct Ops {
    floatx4 a, b;
  } ops[2];
  // (The loads are waited for by count, a chunk after they are issued: no branches around them and one order of issue
  // before and in the loop.  Past the last stage they bring it in again, unused.)
  auto load_a = [&](int d, int s) __attribute__((always_inline)) {
    const int off = 32 * min(s, stages - 1);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int h = 0; h < 2; ++h) ra[d][h] = *reinterpret_cast<const floatx4*>(pa[h] + off);
    __builtin_amdgcn_sched_barrier(0);
  };
  auto load_b = [&](int s) __attribute__((always_inline)) {   // the chunk that begins with stage s
    const int k = min(k_lo + 32 * s + 4 * bc, q.Kp - 4);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int u = 0; u < 2; ++u) rb[u] = *reinterpret_cast<const floatx4*>(pb[u] + k);
    __builtin_amdgcn_sched_barrier(0);
  };
  auto put_b = [&](int buf) __attribute__((always_inline)) {
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      const int r = 8 * u + br;
      *reinterpret_cast<floatx4*>(&Bs[buf][r * KC + 4 * (bc ^ r)]) = rb[u];
    }
  };
  auto put = [&](int d) __attribute__((always_inline)) {
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const int r = 8 * h + lr;
      *reinterpret_cast<floatx4*>(mine + r * 32 + 4 * (lc ^ (r >> 1))) = ra[d][h];
    }
    __builtin_amdgcn_wave_barrier();
  };
  auto get = [&](Ops& o, int buf, int d, int h) __attribute__((always_inline)) {   // slab h of stage d, whose rows of A are in LDS
    o.a = *reinterpret_cast<const floatx4*>(mine + li * 32 + 4 * ((4 * h + lg) ^ (li >> 1)));
    o.b = *reinterpret_cast<const floatx4*>(&Bs[buf][li * KC + 4 * ((8 * d + 4 * h + lg) ^ li)]);
    __builtin_amdgcn_sched_barrier(0);   // (the products of the slab before follow: they cover the way through LDS)
  };
  auto mma = [&](const Ops& o) __attribute__((always_inline)) {
#pragma unroll
    for (int c = 0; c < 4; ++c) acc = __builtin_amdgcn_mfma_f32_16x16x4f32(o.b[c], o.a[c], acc, 0, 0, 0);
  };
  load_b(0);
#pragma unroll
  for (int d = 0; d < D; ++d) load_a(d, d);
  // What the epilogue's own loads depend on.  (Asked for whether it is needed or not, from any readable address then: a
  // branch here, or a comparison, would wait for everything above.)
  const float* const add_src = q.add.src;
  const int* const add_index = q.add.index;
  const int* const gru_has = q.gb.has;
  const double* const tg_delta = q.tg.delta;
  const bool gru = q.gb.dgi != nullptr, tgrad = q.tg.g_w != nullptr;
  const int index_raw = (add_index != nullptr ? add_index : reinterpret_cast<const int*>(A))[add_index != nullptr ? rowc : 0];
  const int has_raw = (gru ? gru_has : reinterpret_cast<const int*>(A))[gru ? rowc : 0];
  const double delta = (tgrad ? tg_delta : reinterpret_cast<const double*>(A))[tgrad ? rowc : 0];
  put_b(0);
  put(0);
  __syncthreads();
  int s0 = 0, buf = 0;
  for (; s0 + D < stages; s0 += D) {
    load_b(s0 + D);
    get(ops[0], buf, 0, 0);
#pragma unroll
    for (int d = 0; d < D; ++d) {   // stage s0 + d; the next slab, or stage, changes its order beside each slab's products
      load_a(d, s0 + d + D);
      get(ops[1], buf, d, 1);
      mma(ops[0]);
      put((d + 1) % D);
      if (d + 1 < D) get(ops[0], buf, d + 1, 0);
      else put_b(buf ^ 1);
      mma(ops[1]);
    }
    buf ^= 1;
    __syncthreads();   // (the buffer that is written next was read before the barrier before)
  }
  // what the epilogue needs, on its way beside the last chunk
  const int arow = add_src == nullptr ? -1 : add_index != nullptr ? index_raw : rowc + q.add.row0, live = N - col;
  const float* const gate = q.add.gate;
  floatx4 e0 = floatx4{0.f, 0.f, 0.f, 0.f}, e1 = e0, e2 = e0, e3 = e0, e4 = e0;
  if (gru) {   // r, z, n, W_hn h + b_hn, h (rows of 16-byte aligned pitch, padded to 32 columns)
    const int ldh = q.gb.ldh, c = min(col, ldh - 4);
    const float* g = q.gb.gates + (size_t)rowc * 4 * ldh + c;
    e0 = *reinterpret_cast<const floatx4*>(g); e1 = *reinterpret_cast<const floatx4*>(g + ldh);
    e2 = *reinterpret_cast<const floatx4*>(g + 2 * ldh); e3 = *reinterpret_cast<const floatx4*>(g + 3 * ldh);
    e4 = *reinterpret_cast<const floatx4*>(q.gb.Hm + (size_t)rowc * ldh + c);
  } else if (!tgrad) {
    if (q.bias != nullptr) e0 = load4(q.bias + col, live, aligned4(q.bias, 0));
    if (arow >= 0) e1 = load4(add_src + (size_t)arow * q.add.ld + col, live, aligned4(add_src, q.add.ld));
    if (gate != nullptr) e2 = load4(gate + (size_t)rowc * q.add.ld_gate + col, live, aligned4(gate, q.add.ld_gate));
  }
  get(ops[0], buf, 0, 0);
#pragma unroll
  for (int d = 0; d < D; ++d)
    if (s0 + d < stages) {
      get(ops[1], buf, d, 1);
      mma(ops[0]);
      if (d + 1 < D) {
        put(d + 1);
        get(ops[0], buf, d + 1, 0);
      }
      if (2 * (s0 + d) + 1 < slabs) mma(ops[1]);
    }

  if (tgrad) {
    // Time-encoding gradient epilogue: the tile is not stored.  Each lane multiplies its row's columns by
    // -sin(w_col delta + b_col) (the argument formed exactly as in the forward kernels); sums over the 16 rows of a
    // wavefront (row rotations) and the four wavefronts (LDS).
    __syncthreads();   // all wavefronts have read their last rows of A
    float (*const red)[4][16] = reinterpret_cast<float (*)[4][16]>(smem);
    floatx4 sw = floatx4{0.f, 0.f, 0.f, 0.f}, sb = sw;
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      if (v < live && row_live) {
        float sn, cs;
        sincos_reduced(fma((double)q.tg.w[col + v], delta, (double)q.tg.b[col + v]), sn, cs);
        sb[v] = -acc[v] * sn;
        sw[v] = sb[v] * (float)delta;
      }
    }
#pragma unroll
    for (int v = 0; v < 4; ++v) { sw[v] = row_sum(sw[v]); sb[v] = row_sum(sb[v]); }
    if (li == 0) {
      *reinterpret_cast<floatx4*>(&red[0][wave][4 * lg]) = sw;
      *reinterpret_cast<floatx4*>(&red[1][wave][4 * lg]) = sb;
    }
    __syncthreads();
    if (tid < 32) {
      const int which = tid >> 4, c = tid & 15;
      if (n0 + c < N)
        atomicAdd((which ? q.tg.g_b : q.tg.g_w) + n0 + c, red[which][0][c] + red[which][1][c] + red[which][2][c] + red[which][3][c]);
    }
    return;
  }
  if (gru) {   // GRU gates backward epilogue: acc is the gradient reaching s' = (1 - z) n + z h
    if (!row_live) return;
    const int dm = q.gb.dm;
    const bool vec = (dm & 3) == 0, has = has_raw != 0;
    float* const gi = q.gb.dgi + (size_t)row * q.gb.ld3 + col;
    float* const gh = q.gb.dgh + (size_t)row * q.gb.ld3 + col;
    floatx4 drp, dzp, dnp, dnr;
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const float ds = acc[v], r = e0[v], z = e1[v], nn = e2[v], hn = e3[v], h = e4[v];
      const float dn = ds * (1.0f - z);
      const float dz = ds * (h - nn);
      const float dp = dn * (1.0f - nn * nn);
      const float dr = dp * hn;
      dnp[v] = has ? dp : 0.f;
      dzp[v] = has ? dz * z * (1.0f - z) : 0.f;
      drp[v] = has ? dr * r * (1.0f - r) : 0.f;
      dnr[v] = has ? dp * r : 0.f;
    }
    store4(gi, drp, live, vec); store4(gi + dm, dzp, live, vec); store4(gi + 2 * dm, dnp, live, vec);
    store4(gh, drp, live, vec); store4(gh + dm, dzp, live, vec); store4(gh + 2 * dm, dnr, live, vec);
    return;
  }
#pragma unroll
  for (int v = 0; v < 4; ++v) {
    const float x = acc[v] + e0[v] + e1[v];
    const bool on = v < live && row_live && (gate == nullptr || e2[v] > 0.f);
    acc[v] = on ? (q.relu ? fmaxf(x, 0.f) : x) : 0.f;
  }
  if (q.colsum != nullptr) {   // column sums of the tile: the wavefront's 16 rows, then one atomic per wavefront and column
    float* cs = q.colsum + (size_t)((row_tile * 4 + wave) & (q.colsum_rows - 1)) * N;
    float sum = 0.f;
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const float t = row_sum(acc[v]);
      sum = li == v ? t : sum;
    }
    if (li < 4 && li < live) atomicAdd(cs + col + li, sum);
  }
  if (row_live) store4(q.C + (size_t)row * q.ldc + col, acc, n_store - col, aligned4(q.C, q.ldc));
}

// ------------------------------------------------------------------------------------------------
// The launches.  Up to two independent problems share one; the second one's workgroups follow the first one's, and after both
// come passengers: write-back scatter + SGD.
// ------------------------------------------------------------------------------------------------
__device__ __forceinline__ int nt_rows_of(const NtGroupPtr gp, int pi) {
  const int* m_dev = gp->p[pi].m_dev;
  return m_dev != nullptr ? min(gp->p[pi].M, load_count(m_dev)) : gp->p[pi].M;
}
__host__ __device__ inline int nt_cols16(int n_store) { return (n_store + 15) >> 4; }
__host__ __device__ inline int nt_row_tiles(int M) { return (M + NT_BM - 1) >> 6; }
static_assert(NT_BM == 64, "the shift above");
__host__ __device__ inline int nt_wgs(int M, int col_tiles) { return col_tiles * ((nt_row_tiles(M) + 7) & ~7); }   // (whole rows of XCDs)

template <int TN>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu((TN == 5 ? 3 : 1), (TN <= 5 ? 4 : 2)))) void gemm_nt_kernel(NtGroup grp) {
  __shared__ __attribute__((aligned(16))) float smem[nt_lds<TN>()];
  warm_kernargs(grp);
  if ((int)blockIdx.x >= grp.gemm_wgs) return wb_sgd_block(grp.tail, blockIdx.x - grp.gemm_wgs);
  const NtGroupPtr gp = (NtGroupPtr)__builtin_amdgcn_kernarg_segment_ptr();
  const int pi = (gp->n > 1 && (int)blockIdx.x >= gp->p[1].wg_begin) ? 1 : 0;
  nt_tile<TN>(gp, pi, (int)blockIdx.x - gp->p[pi].wg_begin, gp->p[pi].col_tiles, nt_rows_of(gp, pi), smem);
}

__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(4, 4))) void gemm_nt_few_kernel(NtGroup grp) {
  __shared__ __attribute__((aligned(16))) float smem[NT_FEW_LDS];
  warm_kernargs(grp);
  if ((int)blockIdx.x >= grp.gemm_wgs) return wb_sgd_block(grp.tail, blockIdx.x - grp.gemm_wgs);
  const NtGroupPtr gp = (NtGroupPtr)__builtin_amdgcn_kernarg_segment_ptr();
  const int pi = (gp->n > 1 && (int)blockIdx.x >= gp->p[1].wg_begin) ? 1 : 0;
  nt_few_tile(gp, pi, (int)blockIdx.x - gp->p[pi].wg_begin, gp->p[pi].col_tiles, nt_rows_of(gp, pi), smem);
}

// Rows that are known on the device only (the problems' m_dev is the same): the kernel for few rows up to NT_FEW_COUNTED tiles,
// tiles of 32 columns beyond, laid out for these.
constexpr int NT_FEW_COUNTED = 512;
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(4, 4))) void gemm_nt_counted_kernel(NtGroup grp) {
  __shared__ __attribute__((aligned(16))) float smem[NT_FEW_LDS > nt_lds<2>() ? NT_FEW_LDS : nt_lds<2>()];
  warm_kernargs(grp);
  if ((int)blockIdx.x >= grp.gemm_wgs) return wb_sgd_block(grp.tail, blockIdx.x - grp.gemm_wgs);
  const NtGroupPtr gp = (NtGroupPtr)__builtin_amdgcn_kernarg_segment_ptr();
  // (no branches: they cost up to 0.4 us.  A problem that is not there has no columns, and begins behind all workgroups)
  const int M = min(gp->p[0].M, load_count(gp->p[0].m_dev)), c0 = nt_cols16(gp->p[0].n_store), c1 = nt_cols16(gp->p[1].n_store);
  const bool few = nt_row_tiles(M) * (c0 + c1) <= NT_FEW_COUNTED;
  const int begin = few ? nt_wgs(M, c0) : gp->p[1].wg_begin, pi = (int)blockIdx.x >= begin ? 1 : 0;   // `begin` of the second problem
  if (few && (int)blockIdx.x >= nt_wgs(M, c0 + c1)) return;
  const int block = (int)blockIdx.x - (pi ? begin : 0);
  if (few) nt_few_tile(gp, pi, block, pi ? c1 : c0, M, smem);
  else nt_tile<2>(gp, pi, block, gp->p[pi].col_tiles, M, smem);
}

// Which kernel, as column blocks of 16 per tile; 0: the one for few rows, NT_COUNTED: on the device.
// Rows known here: by the workgroups of 64 x 16 tiles, in whole rows of XCDs (kernels for few rows / one block / two blocks, us):
//   up to one per compute unit, few rows    roots' output, 544 columns in, 256: 7.4 / 8.3 / 10.9; fewer columns in, up to 0.4 apart
//   up to five, one block                   the same, 384: 10.3 / 9.6 / 11.2; GRU of d_m 200, 608: 14.3 / 13.6 / 13.8, 1,216: 20.3 / 17.7 / 19.7
//   beyond, two blocks                      GRU of d_m 200, 1,824: 26.1 / 23.6 / 22.0, 4,864: 58.4 / 51.3 / 46.6
// With more than 4,096 rows two blocks in any case, and with more than 65,536 wider ones still (less re-reading of A).
// Rows counted on the device, in tiles of 64 x 16 (kernel for few rows / two blocks): GRU of d_m 144, 540: 12.6 / 12.3, 3,500 and
// more: 36 / 28; memory gradient of d_m 200, 273: 15.2 / 16.7, 845: 25.9 / 23.4.  How many there are cannot be told from the
// shapes: a step's 19,800 slots refer to 1,300 nodes on the power-law graphs and to 18,000 on a uniform one.  With up to eight
// column blocks the memory gradient, whose GRU epilogue the kernel for few rows reads and writes 16 bytes at a time, takes that
// one at any count (d_m 100: 7.0 / 11.9 on 600 rows, 34.7 / 37.3 on 19,000), and so does the time-encoding gradient as long as
// there cannot be many rows (d_t 100: 6.2 / 8.4 on 600 rows, 16.6 / 16.0 on 9,500, 34.4 / 32.0 on 28,000; to choose on the device costs
// it 0.7).
constexpr int NT_COUNTED = -1, NT_FEW = 256, NT_ONE = 1280, NT_FEW_TG = 2048;
static int nt_tile_blocks(const NtProblem* p, int n) {
  const int M = p[0].M, rows = p[0].rows_est > 0 ? std::min(p[0].rows_est, M) : M, nb = nt_cols16(p[0].n_store);
  const bool counted = p[0].m_dev != nullptr && (n == 1 || (p[1].m_dev == p[0].m_dev && p[1].M == M));
  if (rows > 65536) {
    int best = 1;
    float best_cost = 1e30f;
    static const int cand[] = {5, 4, 7, 2};
    for (int c : cand) {
      const float cost = (float)(((nb + c - 1) / c) * c) / nb;   // padded / useful columns
      if (cost < best_cost - 1e-6f) { best_cost = cost; best = c; }
    }
    return best;
  }
  int64_t tiles = 0, wgs = 0;
  for (int i = 0; i < n; ++i) {
    tiles += (int64_t)nt_row_tiles(p[i].M) * nt_cols16(p[i].n_store);
    wgs += nt_wgs(p[i].M, nt_cols16(p[i].n_store));
  }
  if (counted) {
    const bool narrow = n == 1 && nb <= 8 && (p[0].gb.dgi != nullptr || (p[0].tg.g_w != nullptr && tiles <= NT_FEW_TG));
    return narrow || tiles <= NT_FEW_COUNTED ? 0 : NT_COUNTED;
  }
  return wgs <= NT_FEW ? 0 : M > 4096 || wgs > NT_ONE ? 2 : 1;
}

void gemm_nt_group(const NtProblem* probs, int n, hipStream_t s, const WbArgs* tail) {
  NtGroup g;
  memset(&g, 0, sizeof(g));
  int tail_blocks = 0;
  if (tail != nullptr) {
    g.tail = *tail;
    tail_blocks = wb_total_blocks(*tail);
  }
  for (int i = 0; i < n && g.n < 2; ++i) {
    NtProblem p = probs[i];
    if (p.M <= 0 || p.N <= 0) continue;
    if (p.n_store < p.N) p.n_store = p.N;
    g.p[g.n++] = p;
  }
  if (g.n == 0 && tail_blocks == 0) return;
  const int tn = g.n > 0 ? nt_tile_blocks(g.p, g.n) : 0, width = tn == NT_COUNTED ? 2 : std::max(tn, 1);
  int total = 0, cols = 0;
  for (int i = 0; i < g.n; ++i) {
    NtProblem& p = g.p[i];
    p.col_tiles = (p.n_store + 16 * width - 1) / (16 * width);
    p.wg_begin = total;
    total += nt_wgs(p.M, p.col_tiles);
    cols += nt_cols16(p.n_store);
  }
  if (tn == NT_COUNTED)   // (with few rows: the workgroups of NT_FEW_COUNTED tiles, in whole rows of XCDs)
    total = std::max(total, cols * ((NT_FEW_COUNTED / cols + 7) & ~7));
  g.gemm_wgs = total;
  if (g.n == 1) g.p[1].wg_begin = total;
  total += tail_blocks;
#define TGNN_NT_CASE(TNV) \
  case TNV: hipLaunchKernelGGL(gemm_nt_kernel<TNV>, dim3(total), dim3(256), 0, s, g); break
  switch (tn) {
    TGNN_NT_CASE(7);
    TGNN_NT_CASE(5);
    TGNN_NT_CASE(4);
    TGNN_NT_CASE(2);
    TGNN_NT_CASE(1);
    case NT_COUNTED: hipLaunchKernelGGL(gemm_nt_counted_kernel, dim3(total), dim3(256), 0, s, g); break;
    default: hipLaunchKernelGGL(gemm_nt_few_kernel, dim3(total), dim3(256), 0, s, g);
  }
#undef TGNN_NT_CASE
}

void gemm_nt(const float* A, int lda, const float* B, int ldb, const float* bias, float* C, int ldc, int M, int N,
             int Kp, int n_store, bool relu, hipStream_t s, const RowAdd& add) {
  const NtProblem p = nt_problem(A, lda, B, ldb, bias, C, ldc, M, N, Kp, n_store, relu, nullptr, add);
  gemm_nt_group(&p, 1, s);
}

// ------------------------------------------------------------------------------------------------
// TN with accumulation: G[n, k] += sum_m D[m, n] * A[m, k], bias[n] += sum_m D[m, n].
// Both operands are m-major, and the sum runs over m: an operand run of the MFMA is eight rows of one column.  Lane
// (li, lg) takes TD consecutive floats D[m][n0 + TD*li ..] and TA consecutive floats A[m][k0 + TA*li ..] of the eight
// rows m = 32 step + 8 lg + j (sixteen vector loads, a lane group reads one contiguous piece of a row), which is the
// operand run of TD (TA) strided columns n = n0 + TD*i + t (k = k0 + TA*j + u): the transposition happens in the
// lane's own registers while the fp32 values are split into their three bf16 parts (split3.h), nothing is staged in
// LDS and the main loop has no barrier.
// A workgroup of TN_W wavefronts owns a (16 TD) x (16 TA) tile of G (64 x 64 in the bulk, narrower pieces
// at the right and bottom edges so that little of the tile is padding) over a chunk of the rows; its
// wavefronts take the 32-row steps of the chunk in turn, and their partial tiles are added in LDS before one
// float atomic per element goes to memory.  The reduction over m is split over workgroups.
// What bounds it: the operands (190 MB a step of 4,000 events) come from beyond the L2s, once per chunk, and a tile
// re-reads them from its XCD's L2; the six MFMAs per pair of operands are 17 us of the launch.  Weight gradients of a
// 4,000-event step 113 -> 80 us, of a 600-event one 24.0 -> 18.6 us, of the stand-alone backward call 58 -> 49 us
// against fp32 MFMAs on 4-row steps.  Relative error against double over 600 to 2,400 roots: 1.3e-7 to 2.0e-7 for W_v
// and W_o (fp32 MFMA: 1.6e-7 to 2.5e-7).
// The bias gradient rides along as column K of A, which the loader replaces by ones.
// ------------------------------------------------------------------------------------------------
#ifndef TGNN_TN_WAVES
#define TGNN_TN_WAVES 4
#endif
constexpr int TN_W = TGNN_TN_WAVES;   // wavefronts per workgroup
constexpr int TN_STEP = 32;   // rows per step of a wavefront: the depth of one MFMA

__device__ __forceinline__ void tn_piece(int len, int idx, int& off, int& width) {
  const int full = len / TT;
  if (idx < full) { off = idx * TT; width = TT; return; }
  const int r = len - full * TT;
  off = full * TT;
  if (r <= 16) width = 16;
  else if (r <= 32) width = 32;
  else width = TT;
}
// Column window of D that one head of head_n columns is tiled over (its start is rounded down to 16 bytes).
__host__ __device__ inline int tn_head_width(int head_n) { return head_n + 3; }

template <int TD> struct FragT;
template <> struct FragT<1> { typedef float type; };
template <> struct FragT<2> { typedef float type __attribute__((ext_vector_type(2))); };
template <> struct FragT<4> { typedef float type __attribute__((ext_vector_type(4))); };
template <int T> __device__ __forceinline__ float frag_get(const typename FragT<T>::type& f, int i) { return f[i]; }
template <> __device__ __forceinline__ float frag_get<1>(const float& f, int) { return f; }
template <int T> __device__ __forceinline__ void frag_set(typename FragT<T>::type& f, int i, float x) { f[i] = x; }
template <> __device__ __forceinline__ void frag_set<1>(float& f, int, float x) { f = x; }
template <int T> __device__ __forceinline__ typename FragT<T>::type frag_zero() {
  typename FragT<T>::type f;
#pragma unroll
  for (int i = 0; i < T; ++i) frag_set<T>(f, i, 0.f);
  return f;
}

// The MFMA operand run of column t: eight rows of one column, as three bf16 parts.
template <int T> __device__ __forceinline__ Split8 tn_split(const typename FragT<T>::type (&f)[8], int t) {
  return split8(floatx4{frag_get<T>(f[0], t), frag_get<T>(f[1], t), frag_get<T>(f[2], t), frag_get<T>(f[3], t)},
                floatx4{frag_get<T>(f[4], t), frag_get<T>(f[5], t), frag_get<T>(f[6], t), frag_get<T>(f[7], t)});
}

// Where partial-tile element (t, u, v) of lane (li, lg) lives in a reduction buffer: element-major, lane-minor
// (stores of one instruction touch 64 consecutive words), with the lane rotated by 16 u so that the final
// pass, which walks a row of the tile (li and u vary, lg fixed), also touches 64 different words.
template <int TA>
__device__ __forceinline__ int tn_slot(int t, int u, int v, int li, int lg) {
  return ((t * TA + u) * 4 + v) * 64 + ((lg * 16 + li + 16 * u) & 63);
}

template <int TD, int TA>
__device__ __forceinline__ bool tn_tile(const float* __restrict__ D, const float* __restrict__ A, int ldd, int lda, int dw,
                                        int aw, int n_lo, int N, int K, float* p00, float* p01, float* p10, float* p11,
                                        int ld00, int ld01, int ld10, int ld11, int n_split, int k_split, float* bias0,
                                        float* bias1, int M, int m_lo, int m_hi, int n0, int k0, float* lds) {
  typedef typename FragT<TD>::type FD;
  typedef typename FragT<TA>::type FA;
  const bool with_bias = bias0 != nullptr || bias1 != nullptr;   // column K of A reads as ones
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);   // uniform: loop bounds stay scalar
  const int li = lane & 15, lg = lane >> 4;

  floatx4 acc[TD][TA];
#pragma unroll
  for (int t = 0; t < TD; ++t)
#pragma unroll
    for (int u = 0; u < TA; ++u) acc[t][u] = floatx4{0.f, 0.f, 0.f, 0.f};

  // Column offsets are clamped into the row (results of columns >= N or > K are dropped at the end); rows
  // >= m_hi are clamped and D is zeroed there.
  const int c_nom = k0 + TA * li;
  const float* pd = D + min(n0 + TD * li, dw - TD);   // dw, aw: columns that may be read from D, A (<= the pitch)
  const float* pa = A + min(c_nom, aw - TA);
  const bool ones = with_bias && K >= k0 && K < k0 + 16 * TA;
  const int n_steps = (m_hi - m_lo + TN_STEP - 1) / TN_STEP;

  FD fd[8];
  FA fa[8];
  auto load = [&](int step) __attribute__((always_inline)) {   // (past the end: clamped rows, unused)
    const int m = m_lo + TN_STEP * step + 8 * lg;
#pragma unroll
    for (int j = 0; j < 8; ++j) fd[j] = *reinterpret_cast<const FD*>(pd + (size_t)min(m + j, M - 1) * ldd);
#pragma unroll
    for (int j = 0; j < 8; ++j) fa[j] = *reinterpret_cast<const FA*>(pa + (size_t)min(m + j, M - 1) * lda);
  };

  // Steps are not dealt out in advance beyond the first per wavefront: a wavefront that is done with a step claims the
  // next free one from a counter in LDS (the wavefronts of a workgroup share their SIMDs unevenly).
  int* next_step = reinterpret_cast<int*>(lds + (TN_W / 2) * TT * TT);
  auto claim = [&]() __attribute__((always_inline)) {
    int v = 0;
    if (lane == 0) v = atomicAdd(next_step, 1);
    return __builtin_amdgcn_readfirstlane(v);
  };
  int step = wave;
  load(step);
  if (tid == 0) { next_step[0] = TN_W; next_step[1] = 0; }   // (after the first loads are on their way)
  __syncthreads();
  while (step < n_steps) {
    const int nxt = claim();
    if (m_lo + TN_STEP * (step + 1) > m_hi) {   // rows out of range: zeros times whatever A holds
      const int m = m_lo + TN_STEP * step + 8 * lg;
#pragma unroll
      for (int j = 0; j < 8; ++j)
        if (m + j >= m_hi) fd[j] = frag_zero<TD>();
    }
    if (ones) {
#pragma unroll
      for (int u = 0; u < TA; ++u)
        if (c_nom + u == K) {
#pragma unroll
          for (int j = 0; j < 8; ++j) frag_set<TA>(fa[j], u, 1.f);
        }
    }
    Split8 d[TD], a[TA];
#pragma unroll
    for (int t = 0; t < TD; ++t) d[t] = tn_split<TD>(fd, t);
#pragma unroll
    for (int u = 0; u < TA; ++u) a[u] = tn_split<TA>(fa, u);
    // the next step's rows are asked for as soon as the registers are free, and come in beside this step's products
    __builtin_amdgcn_sched_barrier(0);
    step = nxt;
    load(step);
    __builtin_amdgcn_sched_barrier(0);
    // A step's sum is formed from zero, smallest terms first, and added to the running sum once: one rounding of the
    // large sum per 32 rows instead of six.
#pragma unroll
    for (int t = 0; t < TD; ++t) {
      floatx4 part[TA];
#pragma unroll
      for (int q = 0; q < SPLIT_TERMS; ++q)
#pragma unroll
        for (int u = 0; u < TA; ++u)
          part[u] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(d[t].p[split_ta(q)], a[u].p[split_tb(q)],
                                                            q == 0 ? floatx4{0.f, 0.f, 0.f, 0.f} : part[u], 0, 0, 0);
#pragma unroll
      for (int u = 0; u < TA; ++u) acc[t][u] += part[u];
    }
  }

  // Has an operand come by that the split cannot take (split3.h)?  Every sum it enters is NaN: one in D a whole row of the tile,
  // one in A a whole column, so a lane looks at one of its columns and one of its rows.
  float any = 0.f;
#pragma unroll
  for (int t = 0; t < TD; ++t) any += (acc[t][0][0] + acc[t][0][1]) + (acc[t][0][2] + acc[t][0][3]);
#pragma unroll
  for (int u = 1; u < TA; ++u) any += acc[0][u][0];
  if (__builtin_expect(any != any, 0)) next_step[1] = 1;

  // Add the wavefronts' partial tiles in LDS: the lower half of the wavefronts store theirs into a buffer
  // each, the upper half add theirs on top, then every thread sums the buffers for its elements and issues
  // one atomic per element.  acc[t][u][v] of lane (li, lg) is n = TD (4 lg + v) + t, k = TA li + u of the tile.
  constexpr int TW = 16 * TA, TILE = 16 * TD * TW, NB = TN_W / 2;
  float* red = lds + (wave % NB) * TILE;
  if (wave < NB) {
#pragma unroll
    for (int t = 0; t < TD; ++t)
#pragma unroll
      for (int u = 0; u < TA; ++u)
#pragma unroll
        for (int v = 0; v < 4; ++v) red[tn_slot<TA>(t, u, v, li, lg)] = acc[t][u][v];
  }
  __syncthreads();
  if (wave >= NB) {
#pragma unroll
    for (int t = 0; t < TD; ++t)
#pragma unroll
      for (int u = 0; u < TA; ++u)
#pragma unroll
        for (int v = 0; v < 4; ++v) red[tn_slot<TA>(t, u, v, li, lg)] += acc[t][u][v];
  }
  __syncthreads();
  if (__builtin_expect(next_step[1] != 0, 0)) return true;   // the tile is left to tn_again
  constexpr int NT = 64 * TN_W;
#pragma unroll
  for (int i = 0; i < (TILE + NT - 1) / NT; ++i) {
    const int e = tid + i * NT;
    if (TILE % NT != 0 && e >= TILE) break;
    const int tn = e / TW, tk = e % TW;           // position in the tile
    const int n = n0 + tn, k = k0 + tk;
    if (n < n_lo || n >= N || k > K) continue;
    const int slot = tn_slot<TA>(tn % TD, tk % TA, (tn / TD) & 3, tk / TA, tn / (4 * TD));
    float x = 0.f;
#pragma unroll
    for (int b = 0; b < NB; ++b) x += lds[b * TILE + slot];
    // (selects instead of indexing: a dynamically indexed local array would live in scratch memory)
    const bool ns = n >= n_split;
    const int nn = n - (ns ? n_split : 0);
    if (k == K) {
      float* const bias = ns ? bias1 : bias0;
      if (bias != nullptr) atomicAdd(bias + nn, x);
    } else {
      const bool ks = k >= k_split;
      float* base = ns ? (ks ? p11 : p10) : (ks ? p01 : p00);
      const int ld = ns ? (ks ? ld11 : ld10) : (ks ? ld01 : ld00);
      atomicAdd(base + (size_t)nn * ld + (k - (ks ? k_split : 0)), x);
    }
  }
  return false;
}

typedef const TnGroup __attribute__((address_space(4))) * TnGroupPtr;
// The last part of tn_tile for a tile with NaNs among its sums, which are taken again in fp32 over the chunk's rows (one that is
// NaN in fp32 as well ends at its first NaN term); TD, TA: the tile's widths in units of 16; h: the head.  Kept apart from the
// tiles' own last loops, and rolled: in them it costs registers and 0.5 to 1 us of a launch of 11 to 23, this 0.1 to 0.3.
__device__ __forceinline__ void tn_again(TnGroupPtr gp, int pi, int h, int m_lo, int m_hi, int n0, int k0, int TD, int TA, const float* lds, int tid) {
  const auto& q = gp->p[pi];
  const auto& o = q.out;
  const float *D = q.D, *A = q.A;
  float* p00 = o.p[0][0];
  int n_lo = 0, N = q.N, K = q.K;
  if (o.head_k > 0) {
    const int first = h * o.head_n, a0 = first & ~3;
    D += a0;
    A += h * o.head_k;
    p00 += (size_t)a0 * o.ld[0][0];
    n_lo = first - a0; N = n_lo + o.head_n;
    K = o.head_cols;
  }
  const int TW = 16 * TA, TILE = 16 * TD * TW;
#pragma unroll 1
  for (int e = tid; e < TILE; e += 64 * TN_W) {
    const int tn = e / TW, tk = e % TW, n = n0 + tn, k = k0 + tk;
    if (n < n_lo || n >= N || k > K) continue;
    const int slot = ((tn % TD * TA + tk % TA) * 4 + ((tn / TD) & 3)) * 64 + ((tn / (4 * TD) * 16 + tk / TA + 16 * (tk % TA)) & 63);
    float x = 0.f;
#pragma unroll 1
    for (int b = 0; b < TN_W / 2; ++b) x += lds[b * TILE + slot];
    if (x != x) {
      x = 0.f;
#pragma unroll 1
      for (int m = m_lo; m < m_hi && x == x; ++m) x += D[(size_t)m * q.ldd + n] * (k == K ? 1.f : A[(size_t)m * q.lda + k]);
    }
    const int ns = n >= o.n_split, ks = k < K && k >= o.k_split;
    float* out = k == K ? (ns ? o.bias[1] : o.bias[0]) : ns || ks ? o.p[ns][ks] : p00;
    const int nn = n - (ns ? o.n_split : 0);
    if (k == K) { if (out != nullptr) atomicAdd(out + nn, x); }
    else atomicAdd(out + (size_t)nn * o.ld[ns][ks] + (k - (ks ? o.k_split : 0)), x);
  }
}

static_assert(sizeof(TnGroup) <= 4096, "the group travels as a kernel argument");
__global__ __launch_bounds__(64 * TN_W) __attribute__((amdgpu_waves_per_eu(2, 2))) void gemm_tn_kernel(TnGroup grp) {
  // Several independent problems share one launch (all weight gradients of a step): find this workgroup's.
  // The argument block is indexed through the kernel-argument segment itself (scalar loads at a computed
  // offset); indexing the by-value parameter would make the compiler spill the whole block to scratch.
  const TnGroupPtr gp = (TnGroupPtr)__builtin_amdgcn_kernarg_segment_ptr();
  const int xcd = blockIdx.x & 7, pos = blockIdx.x >> 3;
  // (a loop over the problems with its scalar loads one after the other took 5 us before the first row was asked for)
  typedef int int16v __attribute__((ext_vector_type(16)));
  typedef unsigned uint4v __attribute__((ext_vector_type(4)));
  const int16v qb = *reinterpret_cast<const int16v __attribute__((address_space(4)))*>(&gp->plan.qbegin[xcd][0]);
  const uint4v qp = *reinterpret_cast<const uint4v __attribute__((address_space(4)))*>(&gp->plan.qprob[0]);
  int slot = -1, begin = 0, end = 0;
#pragma unroll
  for (int t = 0; t < TN_MAX_GROUP; ++t)
    if (pos >= qb[t]) { slot = t; begin = qb[t]; end = qb[t + 1]; }
  if (slot < 0 || slot >= gp->n || pos >= end) return;   // this XCD's queue is shorter than the longest one
  unsigned word = qp[0];
#pragma unroll
  for (int t = 1; t < 4; ++t)
    if ((slot >> 2) == t) word = qp[t];
  const int pi = (word >> (8 * (slot & 3))) & 255u;
  const int local = pos - begin;
  const auto& q = gp->p[pi];
  unsigned long long mine = 0;
  int chunk_word = 0;
#ifdef __HIP_DEVICE_COMPILE__
  {   // (with the problem's cache lines at once, see warm_kernargs)
    static_assert(sizeof(TnProblem) > 128 && sizeof(TnProblem) <= 192, "three or four lines");
    unsigned d0, d1, d2, d3;
    asm volatile("s_load_dword %0, %6, 0x0\n\ts_load_dword %1, %6, 0x40\n\ts_load_dword %2, %6, 0x80\n\ts_load_dword %3, %6, %7\n\t"
                 "s_load_dwordx2 %4, %8, 0x0\n\ts_load_dword %5, %9, 0x0\n\ts_waitcnt lgkmcnt(0)"
                 : "=&s"(d0), "=&s"(d1), "=&s"(d2), "=&s"(d3), "=&s"(mine), "=&s"(chunk_word)
                 : "s"(&gp->p[pi]), "i"(sizeof(TnProblem) - 4), "s"(&gp->plan.mine[xcd][pi]), "s"(&gp->plan.chunks[pi]));
  }
#endif
  const int tiles = q.tiles, chunks = tn_chunks(chunk_word), shift = tn_shift(chunk_word), N = q.N, K = q.K;
  int M = q.M;
  const int* m_dev = q.m_dev;
  float* const bias0 = q.out.bias[0];
  const bool with_bias = bias0 != nullptr || q.out.bias[1] != nullptr;
  const int nth = local / tiles;
  for (int i = 0; i < nth >> shift; ++i) mine &= mine - 1ull;
  if (mine == 0ull) return;   // (never: the queue ends with the last chunk's tiles)
  const int chunk = (__builtin_ctzll(mine) << shift) + (nth & ((1 << shift) - 1));
  int tile = local - nth * tiles;
  if (m_dev != nullptr) M = min(M, load_count(m_dev));   // (the rows there are, split evenly over the launched chunks)
  const int m_chunk = tn_chunk_rows(M, chunks);
  if (chunk * m_chunk >= M) return;   // uniform for the workgroup, before any barrier
  __shared__ __attribute__((aligned(16))) float lds[(TN_W / 2) * TT * TT + 4];   // reduction buffers + step counter
  int m_lo = chunk * m_chunk;
  int m_hi = min(M, m_lo + m_chunk);
  // A problem with per-head blocks is H problems of the same shape side by side: head h multiplies columns
  // [h head_n, (h + 1) head_n) of D with columns [h head_k, h head_k + head_cols) of A.  Its column window of D
  // starts at the 16-byte boundary below the head's first column; the columns in front are not written.
  const float* Dp = q.D;
  const float* Ap = q.A;
  float* p00 = q.out.p[0][0];
  int dw = q.ldd, aw = q.lda, n_lo = 0, n_hi = N, n_tiling = N, Kt = K;
  int h = 0;
  if (q.out.head_k > 0) {
    const int per_head = tiles / q.heads;
    h = tile / per_head;
    tile -= h * per_head;
    const int first = h * q.out.head_n, a0 = first & ~3;
    Dp += a0; dw -= a0;
    Ap += h * q.out.head_k; aw -= h * q.out.head_k;
    p00 += (size_t)a0 * q.out.ld[0][0];
    n_lo = first - a0; n_hi = n_lo + q.out.head_n;
    n_tiling = tn_head_width(q.out.head_n);
    Kt = q.out.head_cols;
  }
  const int Kb = Kt + (with_bias ? 1 : 0);
  const int k_tiles = tn_pieces(Kb);
  const int np = tile / k_tiles, kp = tile - np * k_tiles;
  int n0, wn, k0, wk;
  tn_piece(n_tiling, np, n0, wn);
  tn_piece(Kb, kp, k0, wk);
  bool again = false;
#define TGNN_TN_CASE(WN, WK)                                                                                          \
  if (wn == WN && wk == WK)                                                                                           \
    again = tn_tile<WN / 16, WK / 16>(Dp, Ap, q.ldd, q.lda, dw, aw, n_lo, n_hi, Kt, p00, q.out.p[0][1], q.out.p[1][0],          \
                              q.out.p[1][1], q.out.ld[0][0], q.out.ld[0][1], q.out.ld[1][0], q.out.ld[1][1],            \
                              q.out.n_split, q.out.k_split, bias0, q.out.bias[1], M, m_lo, m_hi, n0, k0, lds);
  TGNN_TN_CASE(64, 64) else TGNN_TN_CASE(64, 32) else TGNN_TN_CASE(64, 16)
  else TGNN_TN_CASE(32, 64) else TGNN_TN_CASE(32, 32) else TGNN_TN_CASE(32, 16)
  else TGNN_TN_CASE(16, 64) else TGNN_TN_CASE(16, 32) else TGNN_TN_CASE(16, 16)
#undef TGNN_TN_CASE
  if (__builtin_expect(again, 0)) tn_again(gp, pi, h, m_lo, m_hi, n0, k0, wn / 16, wk / 16, lds, threadIdx.x);
}

void TnBatch::add(const float* D, int ldd, const float* A, int lda, int M, int N, int K, const OutMap& out,
                  const int* m_dev) {
  // the loader clamps column offsets to ld - 4 and reads whole float4s: pitches below 4 (or below the logical
  // width) would send it out of bounds
  // (K == 0 with a bias output: column sums of D only; A is then any readable matrix of M rows)
  const bool with_bias = out.bias[0] != nullptr || out.bias[1] != nullptr;
  if (M <= 0 || N <= 0 || K < 0 || (K == 0 && !with_bias) || g.n >= TN_MAX_GROUP || ldd < 4 || lda < 4 || (ldd & 3) ||
      (lda & 3) || N > ldd || K > lda)
    return;
  TnProblem& p = g.p[g.n];
  p.D = D; p.ldd = ldd; p.A = A; p.lda = lda; p.M = M; p.N = N; p.K = K;
  if (out.head_k > 0) {   // H problems of head_n x head_cols side by side
    p.heads = N / out.head_n;
    p.tiles = p.heads * tn_pieces(tn_head_width(out.head_n)) * tn_pieces(out.head_cols);
  } else {
    p.heads = 1;
    p.tiles = tn_pieces(N) * tn_pieces(K + (out.bias[0] != nullptr || out.bias[1] != nullptr ? 1 : 0));
  }
  p.m_dev = m_dev; p.out = out;
  g.n++;
}

void TnBatch::launch(hipStream_t s) {
  if (g.n == 0) return;
  TnShape shape[TN_MAX_GROUP];
  for (int i = 0; i < g.n; ++i) {
    const TnProblem& p = g.p[i];
    const bool heads = p.out.head_k > 0, counted = p.m_dev != nullptr;
    // a row count that lives on the device (distinct nodes of a step) is usually a small part of its bound
    shape[i].rows = !counted ? p.M : dev_rows_est > 0 ? std::min(p.M, dev_rows_est) : (p.M + 7) / 8;
    shape[i].counted = counted;
    shape[i].n = heads ? tn_head_width(p.out.head_n) : p.N;
    shape[i].k = (heads ? p.out.head_cols : p.K) + (p.out.bias[0] != nullptr || p.out.bias[1] != nullptr ? 1 : 0);
    shape[i].heads = p.heads;
    shape[i].tiles = p.tiles;
  }
  const int longest = tn_place(g.plan, shape, g.n, tn_chunk_units(shape, g.n) * TN_ROWS);
  hipLaunchKernelGGL(gemm_tn_kernel, dim3(8 * longest), dim3(64 * TN_W), 0, s, g);
  g.n = 0;
}

void gemm_tn_acc(const float* D, int ldd, const float* A, int lda, int M, int N, int K, const OutMap& out,
                 hipStream_t s, const int* m_dev) {
  TnBatch b;
  b.add(D, ldd, A, lda, M, N, K, out, m_dev);
  b.launch(s);
}

}  // namespace tgnn
