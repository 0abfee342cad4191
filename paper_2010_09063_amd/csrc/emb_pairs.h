// Embedding networks: (token, example) pairs instead of (token, step) lists.
//
// A step's gradient with respect to the embedding row it looked up is summed over the steps of the example that carry
// the same token before anything else happens to it (Section 1, item 2a), so an example contributes at most one row
// per DISTINCT token.  emb_accum_kernel adds the scaled rows of all (token, example) pairs into the embedding's
// clipped sum.  Its workgroup w owns the tokens v with v mod n_wg = w -- consecutive token ids, which are the frequent
// ones, go to different workgroups, and a token has at most one pair per example, so the longest list is `batch` pairs
// however often the token occurs -- and keeps their rows in LDS.  An example's pairs are sorted by owner, and a table
// [owner][example] says which of them are whose, so a workgroup reads one row of the table, an example per lane, and
// then only its own pairs.  (Looking through every example's list for them instead is bound by instructions: 32 us at
// 512 examples of 131 pairs.  With the table as [example][owner] every lane reads a cache line of its own: 20 us.)
//
// What that replaces is a counting sort of all batch x steps by token (zero fill, count, scan, fill: 64 us at 131,072
// steps, partly beside the forward pass) and a segmented sum over the lists (31 us).  On the embedding network at 512
// examples x 256 steps (10,000 x 16 table) the two launches below take 10 + 16 us, and the step 136 -> 26 us.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "kernels_seq.h"

// pair = row << 11 | number of steps that carry the token (1 .. 1024); tokens are below 2^21 and token v is row
// v >> wg_shift of workgroup v mod (1 << wg_shift)
#define EMB_PAIR_SHIFT 11
#define EMB_PAIR_COUNT 2047u
#define EMB_WG_MAX 1024 // workgroups that share the tokens

// sort key of step i: owner, row, step
__device__ __forceinline__ uint32_t emb_pair_key(uint32_t v, int i, int wg_shift) {
  return ((v & ((1u << wg_shift) - 1)) << (21 - wg_shift) | v >> wg_shift) << 10 | (uint32_t)i;
}

// Sorted keys in key[0, T): writes the example's pairs and its column of the table (first pair | one past the last << 16
// of owner w at off[w * off_ld]); sq (one value per thread) receives this thread's share of the sum of squared counts.
// head, start [EMB_WG_MAX + 1], wsum: LDS scratch.
template <int KPT>
__device__ __forceinline__ int emb_write_pairs(const uint32_t *key, uint16_t *head, uint16_t *start, int *wsum, int T, int tid,
                                                int wg_shift, uint32_t *__restrict__ pairs, uint32_t *__restrict__ off,
                                                long off_ld, int &sq) {
  const int lane = tid & 63, wave = tid >> 6;
  uint64_t mine[KPT];
#pragma unroll
  for (int m = 0; m < KPT; ++m) {
    const int p = (m << 8) + (tid & 255); // (threads past the first 256 have no part in this)
    const bool h = p < T && (p == 0 || (key[p] >> 10) != (key[p - 1] >> 10));
    mine[m] = __ballot(h);
    if (lane == 0 && wave < 4) wsum[m * 4 + wave] = __popcll(mine[m]);
  }
  __syncthreads();
  int total = 0;
#pragma unroll
  for (int q = 0; q < KPT * 4; ++q) total += wsum[q];
#pragma unroll
  for (int m = 0; m < KPT; ++m) {
    int base = 0;
#pragma unroll
    for (int q = 0; q < KPT * 4; ++q) base += q < m * 4 + wave ? wsum[q] : 0;
    if (wave < 4 && ((mine[m] >> lane) & 1)) head[base + __popcll(mine[m] & ((1ull << lane) - 1))] = (uint16_t)((m << 8) + tid);
  }
  __syncthreads();
  sq = 0;
  for (int r = tid; r < total; r += blockDim.x) {
    const int p = head[r], q = r + 1 < total ? head[r + 1] : T, c = q - p;
    pairs[r] = ((key[p] >> 10) & ((1u << (21 - wg_shift)) - 1)) << EMB_PAIR_SHIFT | (uint32_t)c;
    sq += c * c;
  }
  // first pair of every owner: the number of pairs whose owner is smaller
  const int n_wg = 1 << wg_shift;
  for (int w = tid; w <= n_wg; w += blockDim.x) {
    int lo = 0, hi = total;
    while (lo < hi) {
      const int mid = (lo + hi) >> 1;
      if ((int)(key[head[mid]] >> (31 - wg_shift)) < w) lo = mid + 1; else hi = mid;
    }
    start[w] = (uint16_t)lo;
  }
  __syncthreads();
  for (int w = tid; w < n_wg; w += blockDim.x) off[w * off_ld] = (uint32_t)start[w] | (uint32_t)start[w + 1] << 16;
  return total;
}

// ---------------------------------------------------------------- embedding, mean over the steps, dense classifier
//
// Everything that belongs to one example in one workgroup: the mean of its rows, logits, loss gradient, both layers'
// norms, the clip factor, and what the batch sums need: the mean, s * delta, the row s * (W delta) / T that every step
// of the example passes to its token, and the example's pairs.  The embedding layer's gradient is that one row times
// the number of steps with the token, so its squared norm is |W delta / T|^2 times the sum of the squared counts.
// Bound by latency (T + 4 row loads, a 256-key sort in registers, six barriers), so several workgroups share a CU.
struct BagArgs {
  const int *tok; // [B][T], or the whole dataset where the minibatch is drawn here (draw_n > 0 examples; key draw_k0, draw_k1)
  const float *E, *W, *bias; // [V][D], [D][N], [N]
  const int *y;
  float *mean;     // [B][D]
  float *sdelta;   // [B][16]
  float *rows;     // [B][D]
  uint32_t *pairs; // [B][T]
  uint32_t *off; long off_ld; // [1 << wg_shift][off_ld]
  float *norms, *s; // [B] or null (then nothing is clipped)
  int T, D, N, wg_shift;
  float C;
  long draw_n; uint32_t draw_k0, draw_k1;
};

// DPSGD item 1: index k of the minibatch = (word k % 4 of the Philox block with counter (k / 4, 0, 1, 0)) * n >> 32 --
// uniform over [0, n), with replacement; the third counter word keeps these blocks apart from the noise stream's.
__device__ __forceinline__ long draw_index(int k, long n, uint32_t k0, uint32_t k1) {
  uint32_t r[4];
  philox4x32_10((uint32_t)(k >> 2), 0u, 1u, 0u, k0, k1, r);
  const uint32_t w = k & 2 ? (k & 1 ? r[3] : r[2]) : (k & 1 ? r[1] : r[0]);
  return (long)(((uint64_t)w * (uint64_t)n) >> 32);
}

#define BAG_DMAX 128

template <int KPT, bool VEC>
__global__ __launch_bounds__(256) void bag_net_kernel(const BagArgs a) {
  constexpr int W_ = VEC ? 4 : 1;
  __shared__ uint32_t key[KPT * 256];
  __shared__ uint16_t head[KPT * 256], start[EMB_WG_MAX + 1];
  __shared__ int wsum[KPT * 4];
  __shared__ float part[256 * W_];
  __shared__ float red[256];
  __shared__ float mean[BAG_DMAX], delta[16], wred[4][2];
  __shared__ int cred[4];
  const int b = blockIdx.x, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int T = a.T, D = a.D, N = a.N;
  const long src = a.draw_n > 0 ? draw_index(b, a.draw_n, a.draw_k0, a.draw_k1) : b;
  const int *tok = a.tok + src * T;
  uint32_t kr[KPT];
#pragma unroll
  for (int m = 0; m < KPT; ++m) {
    const int i = (m << 8) + tid;
    const uint32_t v = (uint32_t)tok[min(i, T - 1)];
    key[i] = v;
    kr[m] = i < T ? emb_pair_key(v, i, a.wg_shift) : 0xFFFFFFFFu;
  }
  __syncthreads();
  // mean of the rows: thread (column group c, step group g)
  const int DW = D / W_, G = 256 / DW, c = tid % DW, g = tid / DW;
  {
    float acc[W_] = {};
    if (g < G) {
      for (int t0 = g; t0 < T; t0 += 4 * G) { // four rows in flight
        float v[4][W_];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          const int t = t0 + u * G;
          const float *row = a.E + (long)key[min(t, T - 1)] * D + c * W_;
          if constexpr (VEC) {
            const float4 q = *reinterpret_cast<const float4 *>(row);
            v[u][0] = q.x; v[u][1] = q.y; v[u][2] = q.z; v[u][3] = q.w;
          } else {
            v[u][0] = *row;
          }
        }
#pragma unroll
        for (int u = 0; u < 4; ++u)
#pragma unroll
          for (int w = 0; w < W_; ++w) acc[w] += t0 + u * G < T ? v[u][w] : 0.f;
      }
#pragma unroll
      for (int w = 0; w < W_; ++w) part[g * D + c * W_ + w] = acc[w];
    }
  }
  __syncthreads();
  const int J = 256 / D; // second level: J threads per coordinate
  {
    const int e = tid % D, j = tid / D;
    float v = 0.f;
    if (j < J) {
      for (int q = j; q < G; q += J) v += part[q * D + e];
      red[j * D + e] = v;
    }
  }
  __syncthreads();
  float sa = 0.f;
  if (tid < D) {
    float v = 0.f;
    for (int j = 0; j < J; ++j) v += red[j * D + tid];
    v /= (float)T;
    mean[tid] = v;
    a.mean[(long)b * D + tid] = v;
    sa = v * v;
  }
  __syncthreads();
  // logits: 16 threads per class
  {
    const int n = tid >> 4, j = tid & 15;
    float z = 0.f;
    if (n < N)
      for (int e = j; e < D; e += 16) z += mean[e] * a.W[e * N + n];
#pragma unroll
    for (int o = 8; o > 0; o >>= 1) z += __shfl_xor(z, o, 16);
    if (j == 0) delta[n] = n < N ? z + a.bias[n] : 0.f;
  }
  __syncthreads();
  float d2 = 0.f; // |delta|^2, in every lane of wave 0
  if (wave == 0) {
    const int n = lane & 15;
    float z = n < N ? delta[n] : -INFINITY, mx = z;
#pragma unroll
    for (int o = 8; o > 0; o >>= 1) mx = fmaxf(mx, __shfl_xor(mx, o, 16));
    const float ex = n < N ? expf(z - mx) : 0.f;
    float se = ex;
#pragma unroll
    for (int o = 8; o > 0; o >>= 1) se += __shfl_xor(se, o, 16);
    const float dn = n < N ? ex * (1.f / se) - (n == a.y[src] ? 1.f : 0.f) : 0.f;
    d2 = dn * dn;
#pragma unroll
    for (int o = 8; o > 0; o >>= 1) d2 += __shfl_xor(d2, o, 16);
    if (lane < 16) delta[n] = dn;
  }
  __syncthreads();
  float row = 0.f;
  if (tid < D) {
    for (int n = 0; n < N; ++n) row += a.W[tid * N + n] * delta[n];
    row /= (float)T;
  }
  float sr = row * row;
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) { sa += __shfl_xor(sa, o, 64); sr += __shfl_xor(sr, o, 64); }
  if (lane == 0) { wred[wave][0] = sa; wred[wave][1] = sr; }
  // the example's distinct tokens
  emb_sort_keys<KPT>(kr, key, tid);
#pragma unroll
  for (int m = 0; m < KPT; ++m) key[(m << 8) + tid] = kr[m];
  __syncthreads();
  int sq;
  (void)emb_write_pairs<KPT>(key, head, start, wsum, T, tid, a.wg_shift, a.pairs + (long)b * T, a.off + b, a.off_ld, sq);
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) sq += __shfl_xor(sq, o, 64);
  if (lane == 0) cred[wave] = sq;
  __syncthreads();
  float s = 1.f;
  if (a.s != nullptr) {
    if (wave == 0) {
      const float na = wred[0][0] + wred[1][0], nr = wred[0][1] + wred[1][1]; // (D <= 128: the first two waves)
      const float n2 = (na + 1.f) * d2 + nr * (float)(cred[0] + cred[1] + cred[2] + cred[3]);
      const float nm = sqrtf(n2);
      if (lane == 0) {
        a.norms[b] = nm;
        red[0] = a.s[b] = fminf(1.f, a.C / nm); // nm == 0: C / 0 = +inf -> 1
      }
    }
    __syncthreads();
    s = red[0];
  }
  if (tid < D) a.rows[(long)b * D + tid] = s * row;
  if (tid < 16) a.sdelta[(long)b * 16 + tid] = s * delta[tid];
}

// ---------------------------------------------------------------- embedding below other layers (the LSTM)
//
// Per example: the steps' gradients dx[b, t, :] summed over the steps of each distinct token into rows[b * T + pair], the
// pairs, and the squared norm of those rows (slot[b], null: not wanted).  Two workgroups of 512 threads share a CU; a group of 32
// lanes walks through every sixteenth token with eight steps' loads in flight (the most frequent token of an example
// has some tens of steps, most have one or two).  Bound by HBM: B T D floats read, about half of them written.
struct EmbRowsArgs {
  const int *tok; const float *dx; // [B][T], [B][T][D]
  float *rows, *slot;
  uint32_t *pairs, *off; long off_ld;
  int T, D, wg_shift;
};
#define EMB_ROWS_THREADS 512

// Its lanes hold W_ coordinates of a row: four that follow each other (VEC), or, with rows that start on 4 bytes, every 32nd:
// in rows of more than 32 coordinates one at a time left the walk waiting for one short load after another (251 wide, 349
// steps, 25 examples: 80 -> 55 us; 107, 315, 16: 41 -> 28).  A token's only step is one load.
template <int KPT, int W_, bool VEC>
__global__ __launch_bounds__(EMB_ROWS_THREADS) void emb_rows_kernel(const EmbRowsArgs a) {
  __shared__ uint32_t key[KPT * 256];
  __shared__ uint16_t head[KPT * 256], start[EMB_WG_MAX + 1];
  __shared__ int wsum[KPT * 4];
  __shared__ float red[EMB_ROWS_THREADS / 64];
  const int b = blockIdx.x, tid = threadIdx.x, T = a.T, D = a.D;
  const int *tok = a.tok + (long)b * T;
  uint32_t kr[KPT];
#pragma unroll
  for (int m = 0; m < KPT; ++m) {
    const int i = (m << 8) + (tid & 255);
    kr[m] = i < T ? emb_pair_key((uint32_t)tok[i], i, a.wg_shift) : 0xFFFFFFFFu;
  }
  // (both halves of the workgroup sort the same keys; the barriers inside count every thread)
  emb_sort_keys<KPT>(kr, key, tid & 255);
#pragma unroll
  for (int m = 0; m < KPT; ++m) key[(m << 8) + (tid & 255)] = kr[m];
  __syncthreads();
  int sq;
  const int total = emb_write_pairs<KPT>(key, head, start, wsum, T, tid, a.wg_shift, a.pairs + (long)b * T, a.off + b, a.off_ld, sq);
  const int sub = tid & 31, grp = tid >> 5;
  const float *dx = a.dx + (long)b * T * D;
  float *rows = a.rows + (long)b * T * D;
  float n2 = 0.f;
  for (int u = grp; u < total; u += EMB_ROWS_THREADS / 32) {
    const int p0 = head[u], p1 = u + 1 < total ? head[u + 1] : T;
    for (int e0 = 0; e0 < D; e0 += 32 * W_) {
      const int e = e0 + (VEC ? sub * W_ : sub);
      auto load = [&](float (&v)[W_], int p) {
        const float *r = dx + (long)(key[p] & 1023u) * D;
        if constexpr (VEC) {
          const float4 q = *reinterpret_cast<const float4 *>(r + (e < D ? e : 0));
          v[0] = q.x; v[1] = q.y; v[2] = q.z; v[3] = q.w;
        } else {
#pragma unroll
          for (int w = 0; w < W_; ++w) v[w] = r[min(e + 32 * w, D - 1)];
        }
      };
      float acc[W_] = {};
      if (p1 - p0 == 1) {
        load(acc, p0);
      } else {
        for (int p = p0; p < p1; p += 8) {
          float v[8][W_];
#pragma unroll
          for (int j = 0; j < 8; ++j) load(v[j], min(p + j, p1 - 1));
#pragma unroll
          for (int j = 0; j < 8; ++j)
#pragma unroll
            for (int w = 0; w < W_; ++w) acc[w] += p + j < p1 ? v[j][w] : 0.f;
        }
      }
      if constexpr (VEC) {
        if (e < D) *reinterpret_cast<float4 *>(rows + (long)u * D + e) = make_float4(acc[0], acc[1], acc[2], acc[3]);
      }
#pragma unroll
      for (int w = 0; w < W_; ++w) {
        if (e + (VEC ? 0 : 32 * w) < D) {
          if constexpr (!VEC) rows[(long)u * D + e + 32 * w] = acc[w];
          n2 = fmaf(acc[w], acc[w], n2);
        }
      }
    }
  }
  if (a.slot == nullptr) return;
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) n2 += __shfl_xor(n2, o, 64);
  if ((tid & 63) == 0) red[tid >> 6] = n2;
  __syncthreads();
  if (tid == 0) {
    float t = 0.f;
#pragma unroll
    for (int w = 0; w < EMB_ROWS_THREADS / 64; ++w) t += red[w];
    a.slot[b] = t;
  }
}

// ---------------------------------------------------------------- the batch sum over the pairs

#define EMB_ACC_THREADS 1024
#define EMB_ACC_CAP 2048        // pairs a workgroup holds at a time
#define EMB_ACC_CLS 32          // outputs of the classifier per workgroup (with all 202 of the LSTM network's in one, it took 60 us)
#define EMB_ACC_CHUNK 16        // pairs of one token that a group of lanes adds up at a time
#define EMB_ACC_LDS (38 * 1024) // per workgroup: the rows of its tokens and three counters for each

struct EmbAccumArgs {
  const uint32_t *pairs, *off; long off_ld; // [B][T], [1 << wg_shift][off_ld]
  // rows: not PER_PAIR: rows[b] times the pair's count (one row per example); PER_PAIR: rows[b * T + pair] times scale[b]
  const float *rows, *scale;
  float *out;                // [V][D], every row written (FINAL: not used)
  FinalWrite fin; long w_off; // FINAL: the network is complete with this launch, the table at coordinate 0, the classifier at w_off
  int B, T, D, V, wg_shift;  // 1 << wg_shift workgroups share the tokens
  int lpm;                   // lanes per pair, a power of two
  // further workgroups (emb_accum_grid): sum_b in[b] (x) s delta[b] and sum_b s delta[b] of a classifier of N classes: its input rows
  // [B][Dc], its loss gradient in rows of 16, and the factors that are not in it yet (null: it carries them)
  const float *mean, *sdelta, *dscale; float *out_w; int N, Dc;
};

static inline int emb_accum_grid(int wg_shift, int Dc, int N) { return (1 << wg_shift) + ((Dc + 1) * N + EMB_ACC_CLS - 1) / EMB_ACC_CLS; }
static inline int emb_accum_lanes(int D) { // lanes per pair
  const int n = (D & 3) == 0 ? D / 4 : D;
  int l = 1;
  while (l < 64 && l < n) l <<= 1;
  return l;
}
static inline size_t emb_accum_lds_bytes(long V, int D, int s) {
  const size_t rows = (size_t)((V + (1l << s) - 1) >> s);
  const size_t bytes = 4 * (rows * D + 3 * rows + 2);
  return bytes < 4 * EMB_ACC_THREADS ? 4 * EMB_ACC_THREADS : bytes; // (the classifier's workgroup reduces 1024 floats there)
}
// log2 of the workgroups for a [V][D] table whose rows have to fit their LDS; -1: too large
static inline int emb_accum_wg_shift(long V, int D) {
  for (int s = 8; (1 << s) <= EMB_WG_MAX; ++s)
    if (emb_accum_lds_bytes(V, D, s) <= EMB_ACC_LDS) return s;
  return -1;
}

// Per pass over at most 1024 examples, one per thread: the pairs that belong here go to LDS and are ranked within their
// token with one integer LDS atomic each; after a scan of the counts, groups of lanes add up chunks of a token's pairs
// in registers.  Only the few tokens with more than one chunk meet in an LDS float atomic: with one such atomic per pair
// and coordinate, which is the obvious way, the kernel spent 15 of its 18 us on them.  The order of a token's pairs
// depends on the order in which the integer atomics retire.
// VEC: D is a multiple of 4 and a lane holds four coordinates (at D = 100 half as many lanes per row, all of a chunk's
// rows in flight: 66 -> 25 us on the LSTM network at 512 examples).
template <bool PER_PAIR, bool VEC, bool FINAL>
__global__ __launch_bounds__(EMB_ACC_THREADS) void emb_accum_kernel(const EmbAccumArgs a) {
  extern __shared__ float acc[];
  __shared__ uint2 list[EMB_ACC_CAP];
  __shared__ uint16_t rank[EMB_ACC_CAP], order[EMB_ACC_CAP];
  __shared__ int wtot[EMB_ACC_THREADS / 64], items;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int n_wg = 1 << a.wg_shift, wg = blockIdx.x, D = a.D, T = a.T;
  if (wg >= n_wg) { // the classifier's sums, EMB_ACC_CLS outputs per workgroup: thread (output o, group of examples g)
    const int Dc = a.Dc, n_out = (Dc + 1) * a.N, o0 = (wg - n_wg) * EMB_ACC_CLS;
    const int ch = min(EMB_ACC_CLS, n_out - o0), G = EMB_ACC_THREADS / ch;
    const int o = o0 + tid % ch, g = tid / ch, e = o / a.N, n = o - e * a.N;
    float v = 0.f;
    for (int b = g; b < a.B && g < G; b += 8 * G) { // eight examples in flight
      float m[8], d[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        const long bb = min(b + u * G, a.B - 1);
        m[u] = a.mean[bb * Dc + min(e, Dc - 1)];
        d[u] = a.sdelta[bb * 16 + n];
        if (a.dscale != nullptr) d[u] *= a.dscale[bb];
      }
#pragma unroll
      for (int u = 0; u < 8; ++u) v += b + u * G < a.B ? (e < Dc ? m[u] * d[u] : d[u]) : 0.f;
    }
    acc[tid] = v;
    __syncthreads();
    if (tid < ch) {
      for (int q = 1; q < G; ++q) v += acc[q * ch + tid];
      if (FINAL) final_write(a.fin, a.w_off + o, v);
      else a.out_w[o] = v;
    }
    return;
  }
  const int n_rows = (a.V + n_wg - 1) >> a.wg_shift;
  int *cnt = (int *)(acc + n_rows * D), *first = cnt + n_rows, *item0 = first + n_rows + 1; // item0: [n_rows + 1]
  for (int i = tid; i < n_rows * D; i += EMB_ACC_THREADS) acc[i] = 0.f;
  const int lpm = a.lpm, sub = lane & (lpm - 1), grp = tid / lpm, n_grp = EMB_ACC_THREADS / lpm;
  int step = EMB_ACC_THREADS;
  for (int b0 = 0; b0 < a.B;) {
    int k0 = 0, n = 0, at, total;
    const int b = b0 + tid;
    for (;; step >>= 1) { // (as many examples as the list has room for; at least two, whatever they hold)
      if (tid < step && b < a.B) {
        const uint32_t both = a.off[wg * a.off_ld + b];
        k0 = both & 0xFFFF; n = (int)(both >> 16) - k0;
      } else {
        n = 0;
      }
      at = n; // inclusive scan over the wave, then the waves before this one
#pragma unroll
      for (int o = 1; o < 64; o <<= 1) {
        const int x = __shfl_up(at, o, 64);
        if (lane >= o) at += x;
      }
      __syncthreads(); // (the last pass is done with the lists and the counters)
      if (lane == 63) wtot[wave] = at;
      __syncthreads();
      total = 0;
      at -= n;
#pragma unroll
      for (int w = 0; w < EMB_ACC_THREADS / 64; ++w) {
        if (w < wave) at += wtot[w];
        total += wtot[w];
      }
      if (total <= EMB_ACC_CAP) break;
    }
    for (int i = tid; i < n_rows; i += EMB_ACC_THREADS) cnt[i] = 0;
    __syncthreads();
    for (int k = 0; k < n; k += 2) { // two loads in flight (most examples have one or two pairs for a workgroup)
      uint32_t en[2];
#pragma unroll
      for (int q = 0; q < 2; ++q) en[q] = a.pairs[(long)b * T + k0 + min(k + q, n - 1)];
#pragma unroll
      for (int q = 0; q < 2; ++q)
        if (k + q < n) {
          list[at + k + q] = make_uint2((en[q] & ~EMB_PAIR_COUNT) | (PER_PAIR ? (uint32_t)(k0 + k + q) : en[q] & EMB_PAIR_COUNT), (uint32_t)b);
          rank[at + k + q] = (uint16_t)atomicAdd(&cnt[en[q] >> EMB_PAIR_SHIFT], 1);
        }
    }
    __syncthreads();
    if (wave == 0) { // exclusive sums of the counts and of the chunks
      const int per = (n_rows + 63) >> 6, lo = min(n_rows, lane * per), hi = min(n_rows, lo + per);
      int x = 0, y = 0;
      for (int i = lo; i < hi; ++i) { x += cnt[i]; y += (cnt[i] + EMB_ACC_CHUNK - 1) / EMB_ACC_CHUNK; }
      int ix = x, iy = y;
#pragma unroll
      for (int o = 1; o < 64; o <<= 1) {
        const int px = __shfl_up(ix, o, 64), py = __shfl_up(iy, o, 64);
        if (lane >= o) { ix += px; iy += py; }
      }
      if (lane == 63) { items = iy; item0[n_rows] = iy; }
      ix -= x; iy -= y;
      for (int i = lo; i < hi; ++i) {
        first[i] = ix; item0[i] = iy;
        ix += cnt[i]; iy += (cnt[i] + EMB_ACC_CHUNK - 1) / EMB_ACC_CHUNK;
      }
    }
    __syncthreads();
    for (int i = tid; i < total; i += EMB_ACC_THREADS) order[first[list[i].x >> EMB_PAIR_SHIFT] + rank[i]] = (uint16_t)i;
    __syncthreads();
    for (int it = grp; it < items; it += n_grp) {
      int lo = 0, hi = n_rows; // the last row whose first item is not past `it` and that has one
      while (hi - lo > 1) {
        const int mid = (lo + hi) >> 1;
        if (item0[mid] <= it) lo = mid; else hi = mid;
      }
      const int p0 = first[lo] + (it - item0[lo]) * EMB_ACC_CHUNK, np = min(EMB_ACC_CHUNK, first[lo] + cnt[lo] - p0);
      constexpr int W_ = VEC ? 4 : 1, IN_FLIGHT = VEC ? EMB_ACC_CHUNK : EMB_ACC_CHUNK / 2;
      for (int e0 = 0; e0 < D; e0 += lpm * W_) {
        const int e = e0 + sub * W_, ec = e < D ? e : 0;
        float sum[W_] = {};
        for (int j0 = 0; j0 < np; j0 += IN_FLIGHT) {
          float v[IN_FLIGHT][W_], f[IN_FLIGHT];
#pragma unroll
          for (int j = 0; j < IN_FLIGHT; ++j) {
            const uint2 en = list[order[p0 + min(j0 + j, np - 1)]];
            f[j] = PER_PAIR ? a.scale[en.y] : (float)(en.x & EMB_PAIR_COUNT);
            const float *r = a.rows + (PER_PAIR ? (long)en.y * T + (en.x & EMB_PAIR_COUNT) : (long)en.y) * D + ec;
            if constexpr (VEC) {
              const float4 q = *reinterpret_cast<const float4 *>(r);
              v[j][0] = q.x; v[j][1] = q.y; v[j][2] = q.z; v[j][3] = q.w;
            } else {
              v[j][0] = *r;
            }
          }
#pragma unroll
          for (int j = 0; j < IN_FLIGHT; ++j)
#pragma unroll
            for (int w = 0; w < W_; ++w) sum[w] += j0 + j < np ? f[j] * v[j][w] : 0.f;
        }
        if (e < D) {
          const bool whole = cnt[lo] <= EMB_ACC_CHUNK;
#pragma unroll
          for (int w = 0; w < W_; ++w) {
            if (whole) acc[lo * D + e + w] += sum[w];
            else unsafeAtomicAdd(&acc[lo * D + e + w], sum[w]);
          }
        }
      }
    }
    b0 += step;
  }
  __syncthreads();
  for (int i = tid; i < n_rows * D; i += EMB_ACC_THREADS) {
    const int r = i / D;
    const long v = ((long)r << a.wg_shift) + wg;
    if (v >= a.V) continue;
    if (FINAL) final_write(a.fin, v * D + (i - r * D), acc[i]);
    else a.out[v * D + (i - r * D)] = acc[i];
  }
}
