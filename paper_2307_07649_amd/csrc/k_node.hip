// Everything of a step that depends on a distinct node only (Sec. 3.2.1 and Eq. 1-6), in two launches: UPDT (state rows
// gathered, GRU, s') and the node part of every projection of x = {s' | static} with the score vectors U = q W_k^c.  As
// five launches (state gather, GRU products, gates, projections, U) the rows went through memory four times and every
// launch paid its own start and tail.
//
// Products run on the bf16 matrix cores with split operands (split3.h).  The weights arrive split, in operand order
// (prologue), straight from the L2 to registers, several slabs ahead, and are the first MFMA operand, so that a lane ends
// up with four consecutive columns of one row and stores 16 bytes.
//
// update   a workgroup takes a tile of 16 to 48 rows and one of `groups` parts of the columns of s'.  A wavefront brings
//          in its share of the rows {mail | Phi | edge feature | memory} and forms Phi (fp32 in LDS), then owns 16 columns
//          and computes their four sums (r, z, W_in x, W_hn h), so that the gates are local to a lane; the wavefronts that
//          the columns leave over take parts of the k range.
// project  a workgroup takes a tile of 16 to 64 rows and one of `groups` parts of the column blocks of P and U; the rows
//          are split once, into LDS, and a wavefront works on two column blocks at a time (an LDS read feeds twelve
//          MFMAs).  U is taken from x through the composite weights W_q^T W_k^c, not from q, so that no column of this
//          launch waits for another.
//
// Measured (MI355X, kernel trace, launch to launch): five launches 37 us for 1,284 rows and 140 us for 11,377 rows
// (d_m = d_t = 100, d_e = 172 / 186); these two 25 and 77 us.
//
// What bounds them: a workgroup that does nothing else draws 50 bytes per cycle from the L2 when every compute unit does (63
// with 32 of them; measured on 0.6 and 1.26 MB that all read over and over), this one beside its gathering and MFMAs 40, so
// one that streams all GRU weights (1.26 MB split, d_m = d_t = 100, d_e = 186) takes 11 to 13 us however few rows it has.  Few rows are therefore spread over all compute units by columns, and many rows are taken in tiles as
// tall as LDS allows, where the MFMAs (5 us per 16 rows) hide the stream.
#include <algorithm>

#include "tgnn_internal.h"
#include "device_math.h"
#include "gru_device.h"
#include "split3.h"
#include "unique_device.h"

namespace tgnn {

constexpr int ND_W = 8;             // wavefronts per workgroup, update
constexpr int ND_MAX_RB = 3;        // row blocks of 16 per tile, update
constexpr int ND_LDS = 156 * 1024;  // LDS a tile may take (of 160 KB; the scan and the row flags use the rest)
constexpr int ND_GRID = 252;        // workgroups of the update at a time: one per compute unit, and room for the passengers
constexpr int ND_MAX_GROUPS = 4;    // column groups of a tile of the update, at most (its rows come in once per group)
constexpr int NP_W = 4;             // wavefronts per workgroup, projections
constexpr int NP_MAX_RB = 4;        // row blocks of 16 per tile, projections
constexpr int NP_MAX_KS = 8;        // k slabs of a node row
constexpr int NP_GRID = 512;        // workgroups of the projections at a time: two per compute unit

// floats per row of the fp32 tile {input slabs | memory slabs}, bytes per row and part of a split row; 16 bytes more than
// the row itself: sixteen rows read at one column then start in different banks
__host__ __device__ inline int node_pitch(int kx, int kh) { return 32 * (kx + kh) + 4; }
__host__ __device__ inline int node_xpb(int kp) { return 64 * kp + 16; }

void node_dims(Dims& d) {
  d.nd_cb = (d.dm + 15) / 16; d.nd_kx = (d.d_in + 31) / 32; d.nd_kh = (d.dm + 31) / 32; d.nd_kp = (d.dx + 31) / 32;
  const int rb = ND_LDS / (16 * 4 * node_pitch(d.nd_kx, d.nd_kh));
  // a wavefront per column block of the memory width; wider nodes, and inputs whose tile does not fit, take the separate
  // launches
  d.nd_rb = d.nd_cb <= ND_W && d.nd_kp <= NP_MAX_KS ? std::min(rb, ND_MAX_RB) : 0;
}

// Row blocks per tile and column groups for n rows (known on the device only).  Where the tiles do not all run at once, those
// left over after the whole rounds are spread over all workgroups by as many column groups (groups2) as there is room for.
struct NodeSplit {
  int rb, groups;
};
struct NodeUnits {
  int groups, whole, groups2, units, full;   // `whole`: units of whole rounds, `full`: their tiles
};
__device__ __forceinline__ NodeUnits node_units(const NodeSplit& sp, int tiles, int grid, int g_max) {
  NodeUnits k{sp.groups, tiles * sp.groups, sp.groups, tiles * sp.groups, 0};
  if (k.units > grid) {
    k.full = k.units / grid * grid / sp.groups;
    k.whole = k.full * sp.groups;
    const int left = tiles - k.full;
    if (left > 0) k.groups2 = max(sp.groups, min(g_max, grid / left));
    k.units = k.whole + left * k.groups2;
  }
  return k;
}
struct NodeUnit {
  int tile, group, groups;
};
__device__ __forceinline__ NodeUnit node_unit(const NodeUnits& k, int u) {
  const bool last = u >= k.whole;
  const int groups = last ? k.groups2 : k.groups, v = last ? u - k.whole : u, t = v / groups;
  return NodeUnit{(last ? k.full : 0) + t, v - t * groups, groups};
}
__device__ __forceinline__ int node_tiles(int n, int rb) { return rb == 1 ? (n + 15) / 16 : rb == 2 ? (n + 31) / 32 : rb == 3 ? (n + 47) / 48 : (n + 63) / 64; }
// Update: the splits from the least time per workgroup to the most; the first whose tiles all run at once is taken (a
// workgroup streams its part of the weights, 13 us / groups, and has 5 us of MFMAs per row block and group, of which the
// longer counts, and 3 us of gathering per row block; figures of d_m = d_t = 100, d_e = 186: wider inputs and memories raise
// the first two alike, so that the order holds, and narrow ones are bound by the gathering, where the splits hardly differ).
// Beyond ND_GRID tallest tiles (12,096 rows with three row blocks) these run in rounds.
// (Spelled out: a table of the splits ends up in memory, at a cold load per entry.)
#define TGNN_ND_SPLIT(RB, G, GRID) \
  if (RB <= rb_max && G <= g_max && node_tiles(n, RB) * G <= GRID) return NodeSplit{RB, G};
__device__ __forceinline__ NodeSplit node_update_split(int n, int rb_max, int g_max) {
  TGNN_ND_SPLIT(1, 4, ND_GRID) TGNN_ND_SPLIT(1, 3, ND_GRID) TGNN_ND_SPLIT(1, 2, ND_GRID) TGNN_ND_SPLIT(2, 2, ND_GRID)
  TGNN_ND_SPLIT(3, 2, ND_GRID) TGNN_ND_SPLIT(2, 1, ND_GRID)
  return NodeSplit{rb_max, 1};
}
// Projections: as many column groups as fill the chip with 16-row tiles, then taller tiles (their weights come in less
// often, but a workgroup's stores are longer).
__device__ __forceinline__ NodeSplit node_project_split(int n, int rb_max, int g_max) {
  TGNN_ND_SPLIT(1, 8, NP_GRID) TGNN_ND_SPLIT(1, 6, NP_GRID) TGNN_ND_SPLIT(1, 4, NP_GRID) TGNN_ND_SPLIT(2, 6, NP_GRID)
  TGNN_ND_SPLIT(2, 4, NP_GRID) TGNN_ND_SPLIT(2, 3, NP_GRID) TGNN_ND_SPLIT(2, 2, NP_GRID)
  return NodeSplit{rb_max, g_max < 2 ? 1 : 2};
}
#undef TGNN_ND_SPLIT
__device__ __forceinline__ void node_store4(float* p, const floatx4& v, int live, bool vec) {   // live: columns that exist
  if (live >= 4 && vec) *reinterpret_cast<floatx4*>(p) = v;
  else
    for (int e = 0; e < 4; ++e)
      if (e < live) p[e] = v[e];
}

// The wavefront's 2 NB rows of the tile -> LDS (and, by one group for the backward pass, X and Hm): the rows' ids first, then all of
// their pieces at once (two dependent round trips for all rows together).
template <int NB>
__device__ __forceinline__ void node_gather(const NodeArgs& a, int pitch, bool keep_rows, int n, int row0, float* tile, int* has_s) {
  constexpr int NR = 2 * NB, RL = 4, RM = 2, RE = 4;   // rows per wavefront; 64-wide pieces of mail, memory, edge feature
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  const int my_lr = wave * NR + min(lane, NR - 1), my_row = min(row0 + my_lr, n - 1);
  int my_g = my_row, my_e;
  double my_delta, my_tau = 0.0;
  if (a.gid != nullptr) {
    my_g = a.gid[my_row];
    my_e = a.row_eid[my_row];
    my_delta = a.delta[my_row];
  } else {
    const double mem_ts = a.mem_ts[my_row], mail_ts = a.mail_ts[my_row];
    my_e = a.has_in[my_row] ? my_row : -1;
    my_delta = my_e >= 0 ? mail_ts - mem_ts : 0.0;
    my_tau = my_e >= 0 ? mail_ts : mem_ts;
  }
  const int dm = a.dm, dt = a.dt, de = a.de;
  int g[NR], e[NR];
#pragma unroll
  for (int i = 0; i < NR; ++i) {
    g[i] = __builtin_amdgcn_readlane(my_g, i);
    e[i] = __builtin_amdgcn_readlane(my_e, i);
  }
  float rl[NR][RL], rm[NR][RM], re[NR][RE];
#pragma unroll
  for (int i = 0; i < NR; ++i) {
#pragma unroll
    for (int u = 0; u < RL; ++u)
      if (64 * u < 2 * dm) rl[i][u] = a.mail[(size_t)g[i] * 2 * dm + min(lane + 64 * u, 2 * dm - 1)];
#pragma unroll
    for (int u = 0; u < RM; ++u)
      if (64 * u < dm) rm[i][u] = a.mem[(size_t)g[i] * dm + min(lane + 64 * u, dm - 1)];
#pragma unroll
    for (int u = 0; u < RE; ++u) {
      re[i][u] = 0.f;
      if (64 * u < de && e[i] >= 0) re[i][u] = a.efeat[(size_t)e[i] * de + min(lane + 64 * u, de - 1)];
    }
  }
  if (lane < NR) {
    has_s[my_lr] = my_e >= 0;
    if (a.gid == nullptr && keep_rows && row0 + my_lr < n) a.tau[my_row] = my_tau;
  }
  double delta[NR];
#pragma unroll
  for (int i = 0; i < NR; ++i)
    delta[i] = __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(my_delta), i), __builtin_amdgcn_readlane(__double2loint(my_delta), i));
  // the time encoding of the mails (Eq. 1-2), and the zero columns of both slab ranges
  for (int c0 = 0; c0 < dt; c0 += 64) {
    const int c = c0 + lane;
    if (c < dt) {
      const float w = a.time_w[c], b = a.time_b[c];
#pragma unroll
      for (int i = 0; i < NR; ++i) {
        const float v = time_enc(delta[i], w, b);
        tile[(wave * NR + i) * pitch + 2 * dm + c] = v;
        if (keep_rows && a.X != nullptr && row0 + wave * NR + i < n) a.X[(size_t)(row0 + wave * NR + i) * a.ldx + 2 * dm + c] = v;
      }
    }
  }
#pragma unroll
  for (int i = 0; i < NR; ++i) {
    const int lr = wave * NR + i;
    float* t = tile + lr * pitch;
    for (int c = a.d_in + lane; c < 32 * a.kx; c += 64) t[c] = 0.f;
    for (int c = 32 * a.kx + dm + lane; c < 32 * (a.kx + a.kh); c += 64) t[c] = 0.f;
  }
#pragma unroll
  for (int i = 0; i < NR; ++i) {
    const int lr = wave * NR + i, row = row0 + lr;
    float* t = tile + lr * pitch;
    const bool keep = keep_rows && a.X != nullptr && row < n;
    float* X = a.X + (size_t)row * a.ldx;
    float* Hm = a.Hm + (size_t)row * a.ldh;
#pragma unroll
    for (int u = 0; u < RL; ++u) {
      const int c = lane + 64 * u;
      if (c < 2 * dm) { t[c] = rl[i][u]; if (keep) X[c] = rl[i][u]; }
    }
#pragma unroll
    for (int u = 0; u < RM; ++u) {
      const int c = lane + 64 * u;
      if (c < dm) { t[32 * a.kx + c] = rm[i][u]; if (keep) Hm[c] = rm[i][u]; }
    }
    const int c0 = 2 * dm + dt;
#pragma unroll
    for (int u = 0; u < RE; ++u) {
      const int c = lane + 64 * u;
      if (c < de) { t[c0 + c] = re[i][u]; if (keep) X[c0 + c] = re[i][u]; }
    }
    for (int c = 64 * RE + lane; c < de; c += 64) {
      const float v = e[i] >= 0 ? a.efeat[(size_t)e[i] * de + c] : 0.f;
      t[c0 + c] = v;
      if (keep) X[c0 + c] = v;
    }
  }
}

// Sums that came out NaN (see split3.h), taken again in fp32 from the rows and weights in memory.  An operand that the split
// cannot take makes NaN of everything it meets: one in a row all of the row's results, one in the weights a column of every
// row.  A lane that has seen one looks at all of its results once more after its workgroup's last unit.  What that needs waits
// in LDS and is worked out anew: kept in registers through the units, the kernel arguments of code that is hardly ever run
// cost 1.3 us of an 11 us update and 2 us of a 50 us one (scalar registers spilled in the gather), and as a part of the units
// scratch in the update and one wavefront per SIMD less in the projections of wide rows.
typedef const NodeArgs __attribute__((address_space(4))) NodeKernArgs;
struct NodeKept {
  unsigned long long args;   // the kernel-argument segment
  int block, blocks;         // this workgroup's number, and how many take units
};
template <class Blocks> __device__ __forceinline__ void node_keep(NodeKept& kept, Blocks blocks) {
  if (threadIdx.x == 0) kept = NodeKept{(unsigned long long)__builtin_amdgcn_kernarg_segment_ptr(), (int)blockIdx.x, blocks()};
}

// Is one of n numbers NaN?  (Then all that comes of them is, in fp32, too.)
__device__ __forceinline__ bool node_has_nan(const float* x, int n) {
  for (int i = 0; i < n; i += 8) {   // (eight loads at a time)
    bool nan = false;
#pragma unroll
    for (int u = 0; u < 8; ++u) nan |= x[min(i + u, n - 1)] != x[min(i + u, n - 1)];
    if (nan) return true;
  }
  return false;
}
// The four sums of column c of s' of node row `row`: r, z, n from the memory, n from the input (without the biases).
__device__ __forceinline__ floatx4 node_update_plain(const NodeKernArgs& a, int row, int c, int g, int e) {
  const int dm = a.dm, c0 = 2 * dm + a.dt;
  const double delta = a.gid != nullptr ? a.delta[row] : a.mail_ts[row] - a.mem_ts[row];
  floatx4 s = {0.f, 0.f, 0.f, 0.f};
  const float *wr = a.wih + (size_t)c * a.d_in, *wz = wr + (size_t)dm * a.d_in, *wn = wz + (size_t)dm * a.d_in;
#pragma unroll 1
  for (int k = 0; k < a.d_in && s[1] == s[1]; ++k) {   // (z NaN: so is s', whatever the other sums are)
    float x;
    if (k < 2 * dm) x = a.mail[(size_t)g * 2 * dm + k];
    else if (k < c0) x = time_enc(delta, a.time_w[k - 2 * dm], a.time_b[k - 2 * dm]);
    else x = a.efeat[(size_t)e * a.de + k - c0];
    s[0] += x * wr[k]; s[1] += x * wz[k]; s[3] += x * wn[k];
  }
  wr = a.whh + (size_t)c * dm; wz = wr + (size_t)dm * dm; wn = wz + (size_t)dm * dm;
#pragma unroll 1
  for (int k = 0; k < dm && s[1] == s[1]; ++k) {
    const float x = a.mem[(size_t)g * dm + k];
    s[0] += x * wr[k]; s[1] += x * wz[k]; s[2] += x * wn[k];
  }
  return s;
}
// Columns col .. col + live - 1 (at most four) of node row `row`.  A row without a mail has its memory for s'.
__device__ __forceinline__ void node_update_columns(const NodeKernArgs& a, int row, int col, int live) {
  const int g = a.gid != nullptr ? a.gid[row] : row;
  const int e = a.gid != nullptr ? a.row_eid[row] : a.has_in[row] ? row : -1;
  if (e < 0 || node_has_nan(a.mem + (size_t)g * a.dm, a.dm) || node_has_nan(a.mail + (size_t)g * 2 * a.dm, 2 * a.dm) ||
      node_has_nan(a.efeat + (size_t)e * a.de, a.de))
    return;
#pragma unroll 1
  for (int c = col; c < col + min(live, 4); ++c) {
    float* out = a.Xrow + (size_t)row * a.ldxr + c;
    if (*out == *out) continue;
    const floatx4 s = node_update_plain(a, row, c, g, e);
    const int dm = a.dm;
    const float r = sigmoidf_(s[0] + a.bih[c] + a.bhh[c]), z = sigmoidf_(s[1] + a.bih[dm + c] + a.bhh[dm + c]);
    const float hn = s[2] + a.bhh[2 * dm + c], nn = tanhf_(s[3] + a.bih[2 * dm + c] + r * hn);
    *out = (1.0f - z) * nn + z * a.mem[(size_t)g * dm + c];
    if (a.gates != nullptr) {
      float* q = a.gates + (size_t)row * 4 * a.ldh + c;
      q[0] = r; q[a.ldh] = z; q[2 * a.ldh] = nn; q[3 * a.ldh] = hn;
    }
  }
}
// What this thread has stored of its workgroup's units.
__device__ __forceinline__ void node_update_again(const NodeKept& kept, int tid) {
  const NodeKernArgs& a = *(const NodeKernArgs*)kept.args;
  const int n = a.n_dev != nullptr ? min(a.n_max, *a.n_dev) : a.n_max;
  const NodeSplit sp = node_update_split(n, a.rb_max, a.cb);
  const int rb = sp.rb;
  const NodeUnits units = node_units(sp, node_tiles(n, rb), kept.blocks, min(a.cb, ND_MAX_GROUPS));
  const int lane = tid & 63, wave = tid >> 6;
#pragma unroll 1
  for (int u = kept.block; u < units.units; u += kept.blocks) {
    const NodeUnit t = node_unit(units, u);
    if (wave >= (a.cb + t.groups - 1) / t.groups) continue;   // (a column block lies with the first k part's wavefront)
    const int col = (t.group + wave * t.groups) * 16 + 4 * (lane >> 4);
#pragma unroll 1
    for (int m = 0; m < rb; ++m) {
      const int row = (t.tile * rb + m) * 16 + (lane & 15);
      if (row < n && col < a.dm) node_update_columns(a, row, col, a.dm - col);
    }
  }
}
// The node row x that row `row` of the projections has; NULL: zeros.
template <class Args> __device__ __forceinline__ const float* node_x_row(const Args& a, int row) {
  if (a.x_root == nullptr) return a.Xrow + (size_t)row * a.ldxr;
  if (row < a.R) return a.x_root + (size_t)row * a.dx;
  const int sl = row - a.R, r = sl / a.k;
  return sl - r * a.k < a.cnt[r] ? a.x_nbr + (size_t)sl * a.dx : nullptr;
}
__device__ __forceinline__ float node_plain_dot(int dx, const float* x, const float* w, float s) {
#pragma unroll 1
  for (int j = 0; j < dx && s == s; ++j) s += (x != nullptr ? x[j] : 0.f) * w[j];
  return s;
}
// column `col` of P (col < ldp) or column col - ldp of U
__device__ __forceinline__ float node_project_plain(const NodeKernArgs& a, int row, int col) {
  const float* x = node_x_row(a, row);
  const int half = a.ldp >> 1;
  if (col >= a.ldp) {   // U = q W_k^c of its head
    const int u = col - a.ldp, h = u / a.dcp, c = u - h * a.dcp, dh = a.dO / a.H;
    float s = 0.f;
    if (h < a.H && c < a.dc)
#pragma unroll 1
      for (int n = h * dh; n < (h + 1) * dh && s == s; ++n)
        s += node_plain_dot(a.dx, x, a.wq + (size_t)n * a.dq, a.bias_q[n]) * a.wk[(size_t)n * a.dkv + a.dx + c];
    return s;
  }
  const int sec = col >= half, n = col - sec * half, second = n >= a.dO, m = n - second * a.dO;
  if (n >= 2 * a.dO) return 0.f;   // padding
  const float* w = sec ? (second ? a.wo + (size_t)m * (a.dO + a.dx) + a.dO : a.wq + (size_t)m * a.dq)
                       : (second ? a.wv : a.wk) + (size_t)m * a.dkv;
  return node_plain_dot(a.dx, x, w, a.bias_x[col]);
}
__device__ __forceinline__ void node_project_again(const NodeKept& kept, int rb_max, int tid) {
  const NodeKernArgs& a = *(const NodeKernArgs*)kept.args;
  const int n = a.n_dev != nullptr ? min(a.n_max, *a.n_dev) : a.n_max, pairs = (a.ldp + a.ldz) / 32;
  const NodeSplit sp = node_project_split(n, rb_max, (pairs + 1) / 2);
  const int rb = sp.rb;
  const NodeUnits units = node_units(sp, node_tiles(n, rb), kept.blocks, (pairs + 1) / 2);
  const int lane = tid & 63, wave = tid >> 6;
#pragma unroll 1
  for (int u = kept.block; u < units.units; u += kept.blocks) {
    const NodeUnit t = node_unit(units, u);
#pragma unroll 1
    for (int i = 0; i < rb * 8; ++i) {   // row blocks, and the lane's eight columns of a pair of column blocks
      const int row = (t.tile * rb + (i >> 3)) * 16 + (lane & 15);
      if (row >= n) break;
      const float* x = node_x_row(a, row);
      if (x != nullptr && node_has_nan(x, a.dx)) continue;
#pragma unroll 1
      for (int pr = t.group + wave * t.groups; pr < pairs; pr += t.groups * NP_W) {
        const int col = pr * 32 + ((i >> 2) & 1) * 16 + 4 * (lane >> 4) + (i & 3);
        float* o = col < a.ldp ? a.P + (size_t)row * a.ldp + col : a.U + (size_t)row * a.ldz + (col - a.ldp);
        if (*o != *o) *o = node_project_plain(a, row, col);
      }
    }
  }
}

// One unit of the update: tile rows [row0, row0 + 16 NB), column blocks group, group + groups, ...
template <int NB>
__device__ __forceinline__ void node_update_unit(const NodeArgs& a, int n, int row0, int group, int groups, char* lds, int* has_s, float& seen) {
  constexpr int DEPTH = 2;   // weight slabs in flight per wavefront
  static_assert(DEPTH * NB % 2 == 0, "operand buffers alternate");
  const int pitch = node_pitch(a.kx, a.kh);
  float* tile = reinterpret_cast<float*>(lds);
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  const int li = lane & 15, lg = lane >> 4;
  const int per = (a.cb + groups - 1) / groups;          // column blocks per group, and per workgroup
  const int ks = ND_W / per;                             // k parts
  const int kpart = wave / per, cb = group + (wave - kpart * per) * groups;
  const bool active = kpart < ks && cb < a.cb;
  const int dm = a.dm, col = cb * 16 + 4 * lg, live = dm - col;
  const int KT = a.kx + a.kh;
  const int s_lo = KT * kpart / ks, s_hi = KT * (kpart + 1) / ks;
  floatx4 ar[NB], az[NB], an[NB], ai[NB];
#pragma unroll
  for (int m = 0; m < NB; ++m) ar[m] = az[m] = an[m] = ai[m] = floatx4{0.f, 0.f, 0.f, 0.f};
  const uintx4* wp = reinterpret_cast<const uintx4*>(a.Wg) + (size_t)min(cb, a.cb - 1) * KT * 9 * 64 + lane;
  // The loads of a slab are waited for by count, DEPTH slabs after they are issued.  That needs a loop without branches
  // around them and one order of issue before and in the loop (scheduling barriers), or every round waits for everything.
  uintx4 w[DEPTH][9];
  auto load = [&](uintx4 (&r)[9], int s) __attribute__((always_inline)) {
    __builtin_amdgcn_sched_barrier(0);
    const uintx4* p = wp + (size_t)(min(s, KT - 1) * 9) * 64;
#pragma unroll
    for (int q = 0; q < 9; ++q) r[q] = p[q * 64];
    __builtin_amdgcn_sched_barrier(0);
  };
#pragma unroll
  for (int d = 0; d < DEPTH; ++d) load(w[d], s_lo + d);
  floatx4 br, bz, bi, bn;
#pragma unroll
  for (int v = 0; v < 4; ++v) {
    const int c = min(col + v, dm - 1);
    br[v] = a.bih[c] + a.bhh[c]; bz[v] = a.bih[dm + c] + a.bhh[dm + c]; bi[v] = a.bih[2 * dm + c]; bn[v] = a.bhh[2 * dm + c];
  }
  node_gather<NB>(a, pitch, group == 0, n, row0, tile, has_s);
  __syncthreads();
  if (active) {
    const float* pa = tile + li * pitch + 8 * lg;
    auto read = [&](floatx4 (&r)[2], int s, int m) __attribute__((always_inline)) {
      const float* p = pa + m * 16 * pitch + 32 * min(s, KT - 1);
      r[0] = *reinterpret_cast<const floatx4*>(p);
      r[1] = *reinterpret_cast<const floatx4*>(p + 4);
    };
    // Units (slab, row block) in a row.  While the eighteen MFMAs of one are issued, 16 cycles apart, the vector ALU
    // splits the next one's fp32 run and the one after that is read from LDS.
    Split8 x[2];
    floatx4 raw[2];
    read(raw, s_lo, 0);
    x[0] = split8(raw[0], raw[1]);
    read(raw, NB == 1 ? s_lo + 1 : s_lo, NB == 1 ? 0 : 1);
    auto unit = [&](const uintx4 (&r)[9], int s, int m, const Split8& cur, Split8& nxt) __attribute__((always_inline)) {
      if (m == 0 && s == a.kx) {   // the input part of the third sum is complete; from here on the memory part
#pragma unroll
        for (int q = 0; q < NB; ++q) { ai[q] = an[q]; an[q] = floatx4{0.f, 0.f, 0.f, 0.f}; }
      }
      __builtin_amdgcn_sched_barrier(0);
      nxt = split8(raw[0], raw[1]);
      read(raw, s + (m + 2) / NB, (m + 2) % NB);
#pragma unroll
      for (int t = 0; t < SPLIT_TERMS; ++t) {
        ar[m] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, r[split_ta(t)]), cur.p[split_tb(t)], ar[m], 0, 0, 0);
        az[m] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, r[3 + split_ta(t)]), cur.p[split_tb(t)], az[m], 0, 0, 0);
        an[m] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, r[6 + split_ta(t)]), cur.p[split_tb(t)], an[m], 0, 0, 0);
      }
#pragma unroll
      for (int q = 0; q < 18; ++q) {
        __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);   // one MFMA,
        __builtin_amdgcn_sched_group_barrier(0x002, 3, 0);   // three vector ALU instructions
      }
      __builtin_amdgcn_sched_barrier(0);
    };
    auto row_blocks = [&](int d, int s) __attribute__((always_inline)) {
#pragma unroll
      for (int m = 0; m < NB; ++m) unit(w[d], s, m, x[(d * NB + m) & 1], x[(d * NB + m + 1) & 1]);
    };
    int s0 = s_lo;
    for (; s0 + 2 * DEPTH <= s_hi; s0 += DEPTH) {
#pragma unroll
      for (int d = 0; d < DEPTH; ++d) {
        row_blocks(d, s0 + d);
        load(w[d], s0 + d + DEPTH);
      }
    }
#pragma unroll
    for (int d = 0; d < DEPTH; ++d) {   // the last DEPTH .. 2 DEPTH - 1 slabs (fewer only if the part has fewer)
      if (s0 + d < s_hi) row_blocks(d, s0 + d);
      if (s0 + d + DEPTH < s_hi) load(w[d], s0 + d + DEPTH);
    }
#pragma unroll
    for (int d = 0; d < DEPTH - 1; ++d)
      if (s0 + d + DEPTH < s_hi) row_blocks(d, s0 + d + DEPTH);
    if (s_hi <= a.kx) {   // a k part without memory slabs: its third sum is all input
#pragma unroll
      for (int q = 0; q < NB; ++q) { ai[q] = an[q]; an[q] = floatx4{0.f, 0.f, 0.f, 0.f}; }
    }
  }
  floatx4 h[NB];
#pragma unroll
  for (int m = 0; m < NB; ++m) h[m] = *reinterpret_cast<const floatx4*>(tile + (m * 16 + li) * pitch + 32 * a.kx + min(col, 32 * a.kh - 4));
  if (ks > 1) {   // the k parts meet in LDS, over the tile
    __syncthreads();
    floatx4* red = reinterpret_cast<floatx4*>(lds) + lane;
    if (active && kpart > 0) {
      floatx4* o = red + (wave - per) * 4 * NB * 64;
#pragma unroll
      for (int m = 0; m < NB; ++m) { o[(4 * m) * 64] = ar[m]; o[(4 * m + 1) * 64] = az[m]; o[(4 * m + 2) * 64] = an[m]; o[(4 * m + 3) * 64] = ai[m]; }
    }
    __syncthreads();
    if (active && kpart == 0) {
      for (int k = 1; k < ks; ++k) {
        const floatx4* o = red + (wave + (k - 1) * per) * 4 * NB * 64;
#pragma unroll
        for (int m = 0; m < NB; ++m) { ar[m] += o[(4 * m) * 64]; az[m] += o[(4 * m + 1) * 64]; an[m] += o[(4 * m + 2) * 64]; ai[m] += o[(4 * m + 3) * 64]; }
      }
    }
  }
  if (active && kpart == 0) {   // gates (Eq. 3): lane (li, lg) holds columns col .. col + 3 of row li of each block
#pragma unroll
    for (int m = 0; m < NB; ++m) {
      const int lr = m * 16 + li, row = row0 + lr;
      const bool has = has_s[lr] != 0;
      floatx4 r, z, nn, hn, out;
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        r[v] = sigmoidf_(ar[m][v] + br[v]);
        z[v] = sigmoidf_(az[m][v] + bz[v]);
        hn[v] = an[m][v] + bn[v];
        nn[v] = tanhf_(ai[m][v] + bi[v] + r[v] * hn[v]);
        out[v] = has ? (1.0f - z[v]) * nn[v] + z[v] * h[m][v] : h[m][v];
      }
      if (row < n) {
        if (a.gates != nullptr && has) {   // (columns d_m .. of a block are padding)
          float* g = a.gates + (size_t)row * 4 * a.ldh + col;
          *reinterpret_cast<floatx4*>(g) = r; *reinterpret_cast<floatx4*>(g + a.ldh) = z;
          *reinterpret_cast<floatx4*>(g + 2 * a.ldh) = nn; *reinterpret_cast<floatx4*>(g + 3 * a.ldh) = hn;
        }
        node_store4(a.Xrow + (size_t)row * a.ldxr + col, out, live, (a.ldxr & 3) == 0);
        seen += out[0] + out[1] + out[2] + out[3];   // (columns past d_m: no NaN of their own)
      }
    }
  }
  if (a.ds > 0 && group == 0) {   // static node memory (Sec. 3.1): columns d_m .. of the node row
    for (int i = threadIdx.x; i < 16 * NB * a.ds; i += 64 * ND_W) {
      const int lr = i / a.ds, c = i - lr * a.ds, row = row0 + lr;
      if (row < n) a.Xrow[(size_t)row * a.ldxr + dm + c] = a.stat[(size_t)(a.gid[row] % a.N) * a.ds + c];
    }
  }
}

// Biases of U from those of q: a thread per column.
__host__ __device__ __forceinline__ int node_bias_blocks(const NodeArgs& a) { return (a.H * a.dc + 64 * ND_W - 1) / (64 * ND_W); }
__device__ __forceinline__ void node_bias_block(const NodeArgs& a, int block) {
  const int i = block * 64 * ND_W + threadIdx.x;
  if (i >= a.H * a.dc) return;
  const int h = i / a.dc, c = i - h * a.dc, dh = a.dO / a.H;
  float acc = 0.f;
#pragma unroll 10
  for (int d = 0; d < dh; ++d) acc += a.wk[(size_t)(h * dh + d) * a.dkv + a.dx + c] * a.bias_q[h * dh + d];
  a.bias_u[h * a.dcp + c] = acc;
}
__global__ __launch_bounds__(64 * ND_W) void node_bias_kernel(NodeArgs a) { node_bias_block(a, blockIdx.x); }

__global__ __launch_bounds__(64 * ND_W) void node_update_kernel(NodeArgs a) {
  extern __shared__ __attribute__((aligned(16))) char lds[];
  warm_kernargs_and_grid(a);
  __shared__ int has_s[16 * ND_MAX_RB];
  if (a.epoch_bump != nullptr && blockIdx.x == 0 && threadIdx.x == 0) *a.epoch_bump += 1ull;   // nothing here reads it
  // The last blocks are passengers: the scan of the slot sort and the biases of U.  (Behind the units, in the code too: a
  // jump over their code is a cold instruction-cache line for every workgroup.)
  if (__builtin_expect((int)blockIdx.x >= a.unit_blocks, 0)) {
    const int extra = blockIdx.x - a.unit_blocks;
    if (a.bias_u != nullptr && extra < node_bias_blocks(a)) node_bias_block(a, extra);
    else uniq_scan_block(a.scan);
    return;
  }
  const int n = a.n_dev != nullptr ? min(a.n_max, *a.n_dev) : a.n_max;
  const NodeSplit sp = node_update_split(n, a.rb_max, a.cb);
  const NodeUnits units = node_units(sp, node_tiles(n, sp.rb), a.unit_blocks, min(a.cb, ND_MAX_GROUPS));
  __shared__ NodeKept kept;
  node_keep(kept, [&] { return a.unit_blocks; });
  bool again = false;
  float seen = 0.f;
  for (int u = blockIdx.x; u < units.units; u += a.unit_blocks) {
    const NodeUnit t = node_unit(units, u);
    if (again) __syncthreads();   // the unit before is done with the LDS
    again = true;
    if (sp.rb == 1) node_update_unit<1>(a, n, t.tile * 16, t.group, t.groups, lds, has_s, seen);
    else if (sp.rb == 2) node_update_unit<2>(a, n, t.tile * 32, t.group, t.groups, lds, has_s, seen);
    else node_update_unit<3>(a, n, t.tile * 48, t.group, t.groups, lds, has_s, seen);
  }
  if (__builtin_expect(seen != seen, 0)) node_update_again(kept, threadIdx.x);
}

// ---------------------------------------------------------------------------------------------------------
// Rows row0 .. of x -> three bf16 parts in LDS, zero beyond d_x; from ws.Xrow, or (tgnn_temporal_attn_fwd) from the
// caller's rows, which are then also left in ws.Xrow.
template <int RB, int KS>
__device__ __forceinline__ void node_split_rows(const NodeArgs& a, int n, int row0, char* lds, bool keep) {
  const int xpb = node_xpb(a.kp), part = 16 * RB * xpb;
  const int chunks = 8 * a.kp, total = 16 * RB * chunks;   // runs of four columns per row (at most 64) and per tile (at most 4,096)
  const unsigned magic = ((1u << 22) + chunks - 1) / chunks;   // i / chunks = i magic >> 22 for all i < 4,096
  auto put = [&](const floatx4& v, int lr, int c) __attribute__((always_inline)) {
    unsigned q[2][3];
    split_pair(v[0], v[1], q[0][0], q[0][1], q[0][2]);
    split_pair(v[2], v[3], q[1][0], q[1][1], q[1][2]);
#pragma unroll
    for (int t = 0; t < 3; ++t) *reinterpret_cast<uint2*>(lds + t * part + lr * xpb + 2 * c) = make_uint2(q[0][t], q[1][t]);
  };
  if (a.x_root != nullptr) {
    for (int i = threadIdx.x; i < total; i += 64 * NP_W) {
      const int lr = (int)((unsigned)i * magic >> 22), c = (i - lr * chunks) * 4, row = min(row0 + lr, n - 1);
      floatx4 v = floatx4{0.f, 0.f, 0.f, 0.f};
      const float* src = node_x_row(a, row);
      if (src != nullptr) {
#pragma unroll
        for (int e = 0; e < 4; ++e)
          if (c + e < a.dx) v[e] = src[c + e];
      }
      if (keep && row0 + lr < n) *reinterpret_cast<floatx4*>(a.Xrow + (size_t)row * a.ldxr + c) = v;
      put(v, lr, c);
    }
    return;
  }
  // Up to four runs at a time (as many as a thread has), asked for before the first of them is split: one by one, a tile of 32
  // rows of 200 columns was seven dependent round trips.  (Pad columns of the node rows are zero.)
  constexpr int U = RB * KS / 2 < 4 ? RB * KS / 2 : 4;
  const float* const x = a.Xrow + (size_t)row0 * a.ldxr;
  const int last = n - 1 - row0;
#pragma unroll 1
  for (int i0 = threadIdx.x; i0 < total; i0 += U * 64 * NP_W) {
    floatx4 v[U];
    int lr[U], c[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int i = min(i0 + u * 64 * NP_W, total - 1);   // (past the tile: its last run once more)
      lr[u] = (int)((unsigned)i * magic >> 22);
      c[u] = (i - lr[u] * chunks) * 4;
      v[u] = *reinterpret_cast<const floatx4*>(x + min(lr[u], last) * a.ldxr + c[u]);
    }
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int u = 0; u < U; ++u) put(v[u], lr[u], c[u]);
  }
}

// One unit of the projections: tile rows [row0, row0 + 16 RB), pairs of column blocks of group `group`.  KS: slabs at
// most.  A slab's registers are asked for again, for the wavefront's next pair, as soon as its MFMAs are issued: the
// weights are a whole pair ahead and no load waits for a store.
template <int RB, int KS>
__device__ __forceinline__ void node_project_unit(const NodeArgs& a, int n, int row0, int group, int groups, char* lds, float& seen) {
  node_split_rows<RB, KS>(a, n, row0, lds, group == 0);
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  const int li = lane & 15, lg = lane >> 4;
  const int xpb = node_xpb(a.kp), part = 16 * RB * xpb;
  const int p_blk = a.ldp / 16, pairs = (p_blk + a.ldz / 16) / 2;   // (both pitches are multiples of 32)
  const int stride = groups * NP_W;
  uintx4 w[KS][6];
  floatx4 bias[2];
  auto load = [&](uintx4 (&r)[6], int pr, int s) __attribute__((always_inline)) {   // (past the end: the last one again, unused)
    const uintx4* p = reinterpret_cast<const uintx4*>(a.Wp) + (size_t)(min(pr, pairs - 1) * 2 * a.kp + min(s, a.kp - 1)) * 3 * 64 + lane;
#pragma unroll
    for (int t = 0; t < 3; ++t) { r[t] = p[t * 64]; r[3 + t] = p[(size_t)(a.kp * 3 + t) * 64]; }
  };
  auto load_bias = [&](int pr) __attribute__((always_inline)) {
    const float* p = a.bias_x + min(pr, pairs - 1) * 32 + 4 * lg;
    bias[0] = *reinterpret_cast<const floatx4*>(p);
    bias[1] = *reinterpret_cast<const floatx4*>(p + 16);
  };
  const int first = group + wave * groups;
  load_bias(first);
#pragma unroll
  for (int s = 0; s < KS; ++s) {
    load(w[s], first, s);
    __builtin_amdgcn_sched_barrier(0);
  }
  __syncthreads();
  const char* px = lds + li * xpb + 16 * lg;
  auto pair = [&](int pr, bool more) __attribute__((always_inline)) {
    floatx4 acc[RB][2];
#pragma unroll
    for (int m = 0; m < RB; ++m) { acc[m][0] = bias[0]; acc[m][1] = bias[1]; }
#pragma unroll
    for (int s = 0; s < KS; ++s) {
      if (s < a.kp) {
#pragma unroll
        for (int m = 0; m < RB; ++m) {
          bf16x8 xr[3];
#pragma unroll
          for (int t = 0; t < 3; ++t) xr[t] = *reinterpret_cast<const bf16x8*>(px + t * part + m * 16 * xpb + 64 * s);
#pragma unroll
          for (int t = 0; t < SPLIT_TERMS; ++t) {
            acc[m][0] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, w[s][split_ta(t)]), xr[split_tb(t)], acc[m][0], 0, 0, 0);
            acc[m][1] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, w[s][3 + split_ta(t)]), xr[split_tb(t)], acc[m][1], 0, 0, 0);
          }
        }
      }
      if (more) {
        __builtin_amdgcn_sched_barrier(0);
        load(w[s], pr + stride, s);
        __builtin_amdgcn_sched_barrier(0);
      }
    }
    if (more) load_bias(pr + stride);
    const bool is_u = 2 * pr >= p_blk;
    float* out = is_u ? a.U + (2 * pr - p_blk) * 16 + 4 * lg : a.P + 2 * pr * 16 + 4 * lg;
    const int ld = is_u ? a.ldz : a.ldp;
    // Every column once and every row once.  (With 64-row tiles after the stores: 45.0 against 46.6 us on 20,000 rows, 43.9 without;
    // with fewer between them: 8.7 against 9.7 us on 1,284.)
    auto look = [&](int m) __attribute__((always_inline)) {
      const floatx4 t = acc[m][0] + acc[m][1];
      seen += m == 0 ? t[0] + t[1] + t[2] + t[3] : acc[m][0][0];
    };
#pragma unroll
    for (int m = 0; m < RB; ++m) {
      const int row = row0 + m * 16 + li;
      if (RB < 4) look(m);
      if (row < n) {
        float* o = out + (size_t)row * ld;
        *reinterpret_cast<floatx4*>(o) = acc[m][0];
        *reinterpret_cast<floatx4*>(o + 16) = acc[m][1];
        if (!is_u && a.dP != nullptr) {
          float* z = a.dP + (o - a.P);
          *reinterpret_cast<floatx4*>(z) = floatx4{0.f, 0.f, 0.f, 0.f};
          *reinterpret_cast<floatx4*>(z + 16) = floatx4{0.f, 0.f, 0.f, 0.f};
        }
      }
    }
    if (RB == 4)
#pragma unroll
      for (int m = 0; m < RB; ++m) look(m);
  };
  int pr = first;
  for (; pr + stride < pairs; pr += stride) pair(pr, true);
  if (pr < pairs) pair(pr, false);
}

// Workgroups of the launch, for the units, the step between them and the second look.  With four slabs from the arguments: gridDim
// takes the compiler to 177 registers instead of 211 and 32.2 instead of 31.2 us on 4,000 events.  With eight slabs from gridDim:
// the argument takes it to 256, with 21 more in memory.
template <int KS> __device__ __forceinline__ int node_project_blocks(const NodeArgs& a) { return KS <= 4 ? a.unit_blocks : (int)gridDim.x; }

// (Told that two wavefronts per SIMD are wanted, the compiler keeps the accumulators in vector registers; left to itself it
// moves them to and from accumulation registers, 300 to 400 instructions in all, and takes a register too many for two
// wavefronts with eight slabs.  1,284 rows: 10.2 -> 8.8 us.)
template <int KS>
__global__ __launch_bounds__(64 * NP_W) __attribute__((amdgpu_waves_per_eu(2, 2))) void node_project_kernel(NodeArgs a) {
  extern __shared__ __attribute__((aligned(16))) char lds[];
  warm_kernargs_and_grid(a);
  const int n = a.n_dev != nullptr ? min(a.n_max, *a.n_dev) : a.n_max;
  const int pairs = (a.ldp + a.ldz) / 32;
  const NodeSplit sp = node_project_split(n, KS <= 4 ? NP_MAX_RB : 2, (pairs + 1) / 2);
  const auto blocks = [&] { return node_project_blocks<KS>(a); };
  const NodeUnits units = node_units(sp, node_tiles(n, sp.rb), blocks(), (pairs + 1) / 2);
  __shared__ NodeKept kept;
  node_keep(kept, blocks);
  bool again = false;
  float seen = 0.f;
  for (int u = blockIdx.x; u < units.units; u += blocks()) {
    const NodeUnit t = node_unit(units, u);
    if (again) __syncthreads();
    again = true;
    if (sp.rb == 1) node_project_unit<1, KS>(a, n, t.tile * 16, t.group, t.groups, lds, seen);
    else if (sp.rb == 2) node_project_unit<2, KS>(a, n, t.tile * 32, t.group, t.groups, lds, seen);
    else if (KS <= 4) node_project_unit<KS <= 4 ? 4 : 2, KS>(a, n, t.tile * 64, t.group, t.groups, lds, seen);
  }
  if (__builtin_expect(seen != seen, 0)) node_project_again(kept, KS <= 4 ? NP_MAX_RB : 2, threadIdx.x);
}

NodeArgs node_args(tgnn_ctx* ctx, const tgnn_params* p, int n_max, const int32_t* n_dev) {
  const Dims& d = ctx->d;
  Ws& w = ctx->w;
  NodeArgs a{};
  a.n_dev = n_dev; a.n_max = n_max; a.N = d.N;
  a.time_w = p->time_w; a.time_b = p->time_b; a.bih = p->gru_bih; a.bhh = p->gru_bhh; a.bias_x = w.bias_x;
  a.tau = w.tau; a.Xrow = w.Xrow; a.P = w.P; a.U = w.Umat;
  a.ldx = d.ldx; a.ldh = d.ldh; a.ldxr = d.ldxr; a.ldp = d.ldp; a.ldz = d.ldz;
  a.Wg = w.Wg_s; a.Wp = w.Wp_s;
  a.wih = p->gru_wih; a.whh = p->gru_whh; a.wq = p->wq; a.wv = p->wv; a.wo = p->wo; a.dq = d.dq;
  a.bias_u = w.bias_x + d.ldp; a.wk = p->wk; a.bias_q = w.bias_x + d.ldkv; a.dkv = d.dkv; a.dO = d.dO; a.dc = d.de + d.dt; a.dcp = d.dcp;
  a.H = d.H;
  a.dm = d.dm; a.dt = d.dt; a.de = d.de; a.ds = d.ds; a.dx = d.dx; a.d_in = d.d_in;
  a.cb = d.nd_cb; a.kx = d.nd_kx; a.kh = d.nd_kh; a.kp = d.nd_kp; a.rb_max = d.nd_rb;
  return a;
}

void node_update(const NodeArgs& args, hipStream_t s) {
  NodeArgs a = args;
  if (a.n_max <= 0) return;
  const int rb = std::min(a.rb_max, (a.n_max + 15) / 16);
  a.rb_max = rb;
  const int lds = std::max(16 * rb * 4 * node_pitch(a.kx, a.kh), (ND_W - 1) * 4 * rb * 1024);   // the tile, or the k parts' sums
  const int units = 4 * ((a.n_max + 15) / 16);   // (as many as a split can make of them)
  (void)hipFuncSetAttribute((const void*)node_update_kernel, hipFuncAttributeMaxDynamicSharedMemorySize, ND_LDS);
  a.unit_blocks = std::min(units, ND_GRID);
  const int passengers = (a.bias_u != nullptr ? node_bias_blocks(a) : 0) + (a.scan.gcnt != nullptr ? 1 : 0);
  hipLaunchKernelGGL(node_update_kernel, dim3(a.unit_blocks + passengers), dim3(64 * ND_W), lds, s, a);
}

void node_bias(const NodeArgs& a, hipStream_t s) {
  hipLaunchKernelGGL(node_bias_kernel, dim3(node_bias_blocks(a)), dim3(64 * ND_W), 0, s, a);
}

void node_project(const NodeArgs& args, hipStream_t s) {
  NodeArgs a = args;
  if (a.n_max <= 0) return;
  const int lds = 3 * 16 * (a.kp <= 4 ? NP_MAX_RB : 2) * node_xpb(a.kp);
  const int units = 8 * ((a.n_max + 15) / 16);
  a.unit_blocks = std::min(units, NP_GRID);   // the whole grid
  const dim3 grid(a.unit_blocks);
  if (a.kp <= 4) hipLaunchKernelGGL(node_project_kernel<4>, grid, dim3(64 * NP_W), lds, s, a);
  else hipLaunchKernelGGL(node_project_kernel<NP_MAX_KS>, grid, dim3(64 * NP_W), lds, s, a);
}

}  // namespace tgnn
