// Forward for a handful of query rows against a long key sequence (decoding:
// see decode_shape()).  The tiled and list kernels give a workgroup 128 query
// rows and one head's whole key sequence; with a few rows that is one
// workgroup per head streaming megabytes of K.  Here the keys are split
// instead, and the path is bound by reading K once from HBM:
//   decode_scores_kernel  grid (key chunks, heads): z_ij = (alpha-1) scale_i <q_i,k_j>/sqrt(d)
//                         (Sec. 2.1 scores, eq. (asentmax) scale) for the visible keys, fp32, to
//                         the workspace, and a word per chunk (pack_cmax);
//   decode_scores_mfma_kernel  the same for several rows on the matrix cores, in blocks of 32 keys: blocks
//                         that the row's largest score rules out are not written;
//   decode_solve_kernel   one workgroup per query row: bound on the row maximum, the keys that can be in the
//                         support (z > max - 1: everything else is zero already at the lowest
//                         possible threshold), the threshold of eq. (entmax) by Newton steps from
//                         that lowest threshold (sum_j [z_j - tau]_+^r - 1 is convex and decreasing
//                         in tau, so the steps rise to the root and never pass it), and
//                         O_i = sum_j p_ij v_j over the support.
#pragma once
#include "common.hip.h"
#include "fwd_sparse.hip.h"

namespace entmax {

// dynamic LDS of decode_scores_kernel: Q rows as in memory, the groups' maxima, a coefficient and a limit per row
inline size_t decode_scores_lds(int Nq, int D, size_t esize) { return (size_t)Nq * (D * esize + (kThreads / 8) * 4 + 12); }
constexpr int kDecodeListCap = 4096;    // support candidates kept in LDS; longer ones are re-read from the score row

struct DecodeArgs {
  Geom g;
  const void* Q;
  const void* K;
  const void* V;
  void* O;
  float* tau;     // [B*H*Nq]
  float* scores;  // [B*H*Nq][nks] workspace; nks = Nk rounded up to 4.  decode_scores_kernel writes the entries
                  // j < row_limit(i), decode_scores_mfma_kernel whole 32-key blocks (-inf beyond the limit) and only those whose bit
                  // is set in their chunk's word: nothing else may be read
  uint32_t* cmax; // [B*H*Nq][nchunks] largest score of each chunk of kDecodeChunk keys and which of its 32-key blocks'
                  // scores were written, see pack_cmax()
  int nks, nchunks;
  int chunks_per_wg;  // decode_scores_mfma_kernel: chunks a workgroup takes (at most kDecodeMfmaChunks)
};

// A chunk's word: the largest visible score rounded down to 16 bits (a bf16 that is not larger) above one bit per
// 32-key block of the chunk whose scores were written (kDecodeChunk / 32 = 16 blocks).
static_assert(kDecodeChunk == 16 * 32, "one bit per 32-key block in the low half of the word");
constexpr uint32_t kCmaxNone = 0xff800000u;  // -inf, nothing written
__device__ __forceinline__ uint32_t pack_cmax(float m, uint32_t written) {
  const uint32_t u = __float_as_uint(m);
  const uint32_t down = (u & 0x80000000u) ? u + 0xffffu : u;  // towards -inf: a negative number's magnitude goes up
  return (m == -kInf ? kCmaxNone : down & 0xffff0000u) | (written & 0xffffu);
}
// a value not above / not below the chunk's largest score
__device__ __forceinline__ float cmax_floor(uint32_t w) { return __uint_as_float(w & 0xffff0000u); }
__device__ __forceinline__ float cmax_ceil(uint32_t w) {
  const float f = cmax_floor(w);
  return fmaf(fabsf(f), 0x1p-7f, f) + 0x1p-126f;  // (one step of a bf16 is at most 2^-7 of its value)
}
// order-preserving map of floats to signed integers, and back
__device__ __forceinline__ int ordered_bits(float x) {
  const int i = __float_as_int(x);
  return i >= 0 ? i : i ^ 0x7fffffff;
}
__device__ __forceinline__ float from_ordered_bits(int i) { return __int_as_float(i >= 0 ? i : i ^ 0x7fffffff); }

// x + (x of the lane that the DPP control CTRL pairs this lane with): one VALU instruction, no LDS traffic.
template <int CTRL>
__device__ __forceinline__ float dpp_add(float x) {
  return x + __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), CTRL, 0xf, 0xf, false));
}
// Sum over each aligned group of eight lanes, in every lane of the group: lane k adds lane 7-k
// (row_half_mirror), then its neighbour in the pair (quad_perm [1,0,3,2]), then the other pair of its quad
// (quad_perm [2,3,0,1]).  The additions form the same tree in all eight lanes, so they agree to the bit.
__device__ __forceinline__ float sum8(float x) {
  x = dpp_add<0x141>(x);
  x = dpp_add<0xB1>(x);
  return dpp_add<0x4E>(x);
}

// Eight lanes share a key row (each a contiguous eighth of its features), so a wave's load
// instruction covers eight whole rows; a thread keeps four rows in flight.
template <typename T, int D>
__global__ __launch_bounds__(kThreads) void decode_scores_kernel(DecodeArgs A) {
  constexpr int kSlice = D / 8;
  extern __shared__ __align__(16) char decode_lds[];
  const Geom& g = A.g;
  constexpr int kRowWords = D * (int)sizeof(T) / 4;
  constexpr int kGroups = kThreads / 8;
  uint32_t* qw = reinterpret_cast<uint32_t*>(decode_lds);                  // [Nq][kRowWords]
  float* group_max = reinterpret_cast<float*>(qw + g.Nq * kRowWords);      // [Nq][kGroups]: entry [i][grp] is touched
                                                                           // by the group's first lane only
  float* coef = group_max + g.Nq * kGroups;                                // [Nq]
  int* limit = reinterpret_cast<int*>(coef + g.Nq);                        // [Nq]
  float* ybias = reinterpret_cast<float*>(limit + g.Nq);                   // [Nq] distance bias per unit distance, times (alpha-1)
  const int tid = threadIdx.x, bh = blockIdx.y, b = bh / g.H, h = bh % g.H;
  const int j0 = blockIdx.x * kDecodeChunk;
  const T* Qh = reinterpret_cast<const T*>(A.Q) + (long long)b * g.q_sb + (long long)h * g.q_sh;
  const T* Kh = reinterpret_cast<const T*>(A.K) + (long long)b * g.kv_sb + (long long)h * g.kv_sh;
  // the first key rows are requested before anything else: their addresses need nothing from the queries
  const int grp = tid >> 3, sub = tid & 7;
  const int jend = min(j0 + kDecodeChunk, g.Nk);
  RawRow<T, kSlice> nx[4];
  auto fetch = [&](RawRow<T, kSlice>* dst, int base) {
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int j = min(base + u * 32 + grp, g.Nk - 1);  // rows past the end repeat the last one and are not written
      dst[u].load(Kh + (long long)j * g.kv_sn + sub * kSlice);
    }
  };
  fetch(nx, j0);
  // Q in LDS as it is in memory: fp32, or bf16 pairs (then row i starts at word i * D/2)
  for (int e = tid; e < g.Nq * kRowWords; e += kThreads) {
    const int i = e / kRowWords, c = e % kRowWords;
    qw[e] = reinterpret_cast<const uint32_t*>(Qh + (long long)i * g.q_sn)[c];
  }
  if (tid < g.Nq) {
    const int lim = row_limit(g, tid);
    limit[tid] = lim;
    for (int w = 0; w < kGroups; ++w) group_max[tid * kGroups + w] = -kInf;
    const float cf = (g.alpha - 1.0f) * row_scale(g, b, h, tid, lim, nullptr, nullptr, nullptr) * (1.0f / sqrtf((float)D));
    coef[tid] = cf;
    // the same product a w as in the tiled kernels (bias_w(): sign taken from the scale)
    ybias[tid] = fabsf(cf) * bias_w<D>(g, h, cf, fabsf(cf));
  }
  __syncthreads();
  for (int base = j0; base < jend; base += 128) {
    RawRow<T, kSlice> kk[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) kk[u] = nx[u];
    if (base + 128 < jend) fetch(nx, base + 128);  // the next rows are on their way during the arithmetic
    for (int i = 0; i < g.Nq; ++i) {
      constexpr int kWords = RawRow<T, kSlice>::kWords;
      u32x4_t qv[kWords];  // the lane's slice of query row i
#pragma unroll
      for (int w = 0; w < kWords; ++w)
        qv[w] = *reinterpret_cast<const u32x4_t*>(&qw[i * kRowWords + sub * (kRowWords / 8) + 4 * w]);
      const float c = coef[i];
      const int lim = limit[i];
      const float yb = ybias[i];
      const int pos = i + (g.Nk - g.Nq);
      float best = -kInf;
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        float dot = 0.f;
#pragma unroll
        for (int w = 0; w < kWords; ++w) {
#pragma unroll
          for (int k = 0; k < 4; ++k) {
            if constexpr (sizeof(T) == 2)
              dot = dot2_bf16(kk[u].w[w][k], qv[w][k], dot);  // two features per instruction, nothing to widen
            else
              dot = fmaf(__uint_as_float(kk[u].w[w][k]), __uint_as_float(qv[w][k]), dot);
          }
        }
        const int j = base + u * 32 + grp;
        const float zj = fmaf(yb, (float)bias_dist(pos, j), sum8(dot) * c);
        if (j < lim) best = fmaxf(best, zj);
        if (sub == u && j < lim) A.scores[((long long)bh * g.Nq + i) * A.nks + j] = zj;
      }
      if (sub == 0) group_max[i * kGroups + grp] = fmaxf(group_max[i * kGroups + grp], best);
    }
  }
  __syncthreads();
  for (int i0 = 0; i0 < g.Nq; i0 += 8) {
    // thread (i, grp) of an 8 x 32 arrangement: the row's maximum over the 32 groups
    const int i = i0 + (tid >> 5);
    float mx = i < g.Nq ? group_max[i * kGroups + (tid & 31)] : -kInf;
#pragma unroll
    for (int off = 16; off >= 1; off >>= 1) mx = fmaxf(mx, __shfl_xor(mx, off));
    if ((tid & 31) == 0 && i < g.Nq) A.cmax[((long long)bh * g.Nq + i) * A.nchunks + blockIdx.x] = pack_cmax(mx, 0xffffu);
  }
}

// The same scores for several query rows on the matrix cores (bf16 from kDecodeMfmaRows rows on, fp32 from
// kDecodeMfmaRowsF32): S^T = K_block Q^T with 32-key blocks whose fragments come straight from global memory (each
// K row is read once, the next block's rows while this one is computed on) against NQB 32-query blocks.  A lane owns
// a query row and 16 of the block's 32 keys, so a row's largest score of the block is 15 maxima and one exchange.
// What bounds it is reading K once; the fp32 scores of 64 rows would be twice the bytes of K.  So a row's scores of a
// block are written only if the largest of them is above the row's largest score so far less one, whatever wave of
// the workgroup found that: a key at or below (largest score) - 1 has probability zero (App. A, lower end of the
// bracket).  Which blocks of a chunk were written is noted beside the chunk's maximum (pack_cmax).  The two lanes of a row
// each write half of a block's scores: the first one decides for both (the row's largest score may change under their reads).
// Measured: 48 heads, 64 rows, 32768 keys, D 64: 156 us with every score written, 57 us so (two blocks on their way
// instead of one: the same); 128 heads, 5 rows, 6007 keys, D 128: 41 us with per-row dot products (5 us a row at 201 MB of
// K), 32 us so, which is 6.1 TB/s on K (read again every time: part of it stays in the last-level cache).
template <typename T, int D, int NQB>
__global__ __launch_bounds__(kThreads) void decode_scores_mfma_kernel(DecodeArgs A) {
  constexpr int NC = D / 16;
  constexpr int kBlocksPerChunk = kDecodeChunk / 32;
  __shared__ int rowmax[NQB * 32];                                   // ordered_bits() of a row's largest score so far
  __shared__ float wmax[kDecodeMfmaChunks][kWaves][NQB * 32];        // per chunk: what each wave saw and wrote
  __shared__ uint32_t wmask[kDecodeMfmaChunks][kWaves][NQB * 32];
  const Geom& g = A.g;
  const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63, li = lane & 31, hh = lane >> 5;
  const int bh = blockIdx.y, b = bh / g.H, h = bh % g.H;
  const int chunk0 = blockIdx.x * A.chunks_per_wg;
  const int nblk = min(A.chunks_per_wg * kBlocksPerChunk, (g.Nk - chunk0 * kDecodeChunk + 31) >> 5);  // 32-key blocks of this workgroup
  const int jc0 = chunk0 * kDecodeChunk;
  const T* Qh = reinterpret_cast<const T*>(A.Q) + (long long)b * g.q_sb + (long long)h * g.q_sh;
  const T* Kh = reinterpret_cast<const T*>(A.K) + (long long)b * g.kv_sb + (long long)h * g.kv_sh;
  Frag<T> kf[NC], kn[NC];
  auto fetch = [&](Frag<T>* dst, int blk) {  // (rows past the end repeat the last one; their scores are masked)
    const T* krow = Kh + (long long)min(jc0 + blk * 32 + li, g.Nk - 1) * g.kv_sn + 8 * hh;
#pragma unroll
    for (int cc = 0; cc < NC; ++cc) dst[cc] = Elem<T>::load(krow + 16 * cc);
  };
  if (wave < nblk) fetch(kn, wave);
  Frag<T> qf[NQB][NC];
  float cf[NQB], yb[NQB], top[NQB], cm[NQB];
  int lim[NQB];
  uint32_t mask[NQB];
#pragma unroll
  for (int qb = 0; qb < NQB; ++qb) {
    const int i = qb * 32 + li;
    const bool valid = i < g.Nq;
    lim[qb] = valid ? row_limit(g, i) : 0;
    cf[qb] = valid ? (g.alpha - 1.0f) * row_scale(g, b, h, i, lim[qb], nullptr, nullptr, nullptr) * (1.0f / sqrtf((float)D)) : 0.f;
    yb[qb] = valid ? fabsf(cf[qb]) * bias_w<D>(g, h, cf[qb], fabsf(cf[qb])) : 0.f;
    top[qb] = cm[qb] = -kInf;
    mask[qb] = 0u;
#pragma unroll
    for (int cc = 0; cc < NC; ++cc)
      qf[qb][cc] = valid ? Elem<T>::load(Qh + (long long)i * g.q_sn + 16 * cc + 8 * hh) : Elem<T>::zero();
  }
  if (tid < NQB * 32) rowmax[tid] = ordered_bits(-kInf);
  for (int e = tid; e < kDecodeMfmaChunks * kWaves * NQB * 32; e += kThreads) {
    (&wmax[0][0][0])[e] = -kInf;
    (&wmask[0][0][0])[e] = 0u;
  }
  // keys before this one take the short way: every row sees them (row 0 sees the fewest) and none carries a bias
  const int plain_end = g.slopes != nullptr && g.slopes[h] != 0.f ? 0 : row_limit(g, 0);
  __syncthreads();
  for (int blk = wave; blk < nblk; blk += kWaves) {
#pragma unroll
    for (int cc = 0; cc < NC; ++cc) kf[cc] = kn[cc];
    if (blk + kWaves < nblk) fetch(kn, blk + kWaves);
    const int j0 = jc0 + blk * 32;
#pragma unroll
    for (int qb = 0; qb < NQB; ++qb) {
      f32x16_t acc = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int cc = 0; cc < NC; ++cc) acc = Elem<T>::mma(kf[cc], qf[qb][cc], acc);
      // acc[4 q + r] of lane l: key j0 + 8 q + 4 (l/32) + r, query qb*32 + l%32
      if (j0 + 32 <= plain_end) {
        // no bias, and every row sees the whole block: nothing to select per score
#pragma unroll
        for (int e = 0; e < 16; ++e) acc[e] *= cf[qb];
      } else {
        const int rel = lim[qb] - j0 - 4 * hh, pos = qb * 32 + li + (g.Nk - g.Nq) - j0 - 4 * hh;
#pragma unroll
        for (int e = 0; e < 16; ++e) {
          const int k = 8 * (e >> 2) + (e & 3);
          const float zj = fmaf(yb[qb], (float)max(pos - k, 0), acc[e] * cf[qb]);
          acc[e] = k < rel ? zj : -kInf;
        }
      }
      float m = max16(acc);
      m = fmaxf(m, __shfl_xor(m, 32));
      cm[qb] = fmaxf(cm[qb], m);
      // (an older value only writes more)
      top[qb] = fmaxf(top[qb], from_ordered_bits(__hip_atomic_load(&rowmax[qb * 32 + li], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP)));
      // (m = -inf for rows that see none of the block; lim = 0 beyond the last row)
      const uint32_t rows = (uint32_t)__ballot(m > top[qb] - 1.0f && lim[qb] > 0);  // as lanes 0 to 31 see it
      if ((rows >> li) & 1u) {
        if (m > top[qb]) {
          top[qb] = m;
          atomicMax(&rowmax[qb * 32 + li], ordered_bits(m));
        }
        mask[qb] |= 1u << (blk % kBlocksPerChunk);
        float* dst = A.scores + ((long long)bh * g.Nq + qb * 32 + li) * A.nks;
#pragma unroll
        for (int q4 = 0; q4 < 4; ++q4) {
          const int j = j0 + 8 * q4 + 4 * hh;
          if (j < A.nks)  // nks and j are multiples of 4
            *reinterpret_cast<f32x4_t*>(dst + j) = f32x4_t{acc[4 * q4], acc[4 * q4 + 1], acc[4 * q4 + 2], acc[4 * q4 + 3]};
        }
      }
      if (blk % kBlocksPerChunk + kWaves >= kBlocksPerChunk || blk + kWaves >= nblk) {  // this wave's last block of the chunk
        if (hh == 0) {
          wmax[blk / kBlocksPerChunk][wave][qb * 32 + li] = cm[qb];
          wmask[blk / kBlocksPerChunk][wave][qb * 32 + li] = mask[qb];
        }
        cm[qb] = -kInf;
        mask[qb] = 0u;
      }
    }
  }
  __syncthreads();
  for (int e = tid; e < A.chunks_per_wg * NQB * 32; e += kThreads) {
    const int c = e / (NQB * 32), i = e % (NQB * 32);
    if (i >= g.Nq || chunk0 + c >= A.nchunks) continue;
    float mx = wmax[c][0][i];
    uint32_t mk = wmask[c][0][i];
#pragma unroll
    for (int w = 1; w < kWaves; ++w) {
      mx = fmaxf(mx, wmax[c][w][i]);
      mk |= wmask[c][w][i];
    }
    A.cmax[((long long)bh * g.Nq + i) * A.nchunks + chunk0 + c] = pack_cmax(mx, mk);
  }
}

// Sum of two values over the workgroup; every thread gets the totals.  `buf` holds 2 * 2 * NT / 64
// floats: calls alternate between its halves (parity), so one barrier per call is enough.
template <int NT>
__device__ __forceinline__ float2 decode_block_sum(float a, float b, float* buf, int parity) {
  constexpr int kW = NT / 64;
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) {
    a += __shfl_xor(a, off);
    b += __shfl_xor(b, off);
  }
  float* mine = buf + parity * 2 * kW;
  if ((threadIdx.x & 63) == 0) {
    mine[threadIdx.x >> 6] = a;
    mine[kW + (threadIdx.x >> 6)] = b;
  }
  __syncthreads();
  float sa = 0.f, sb = 0.f;
#pragma unroll
  for (int w = 0; w < kW; ++w) {
    sa += mine[w];
    sb += mine[kW + w];
  }
  return make_float2(sa, sb);
}

// One Newton step of sum_j [z_j - tau]_+^r = 1 from the sums F = sum x^r, G = sum x^(r-1); true when tau is final.
__device__ __forceinline__ bool decode_newton(float F, float G, float r, float& tau) {
  if (!(G > 0.f)) return true;
  const float step = (F - 1.0f) / (r * G);  // f = F - 1, f' = -r G; G > 0 while tau < max
  if (!(step > 0.f)) return true;
  tau += step;
  return step <= 1e-6f * fmaxf(1.0f, fabsf(tau));  // what is left is a small multiple of the last step
}

// NT threads per row.  The work of a typical row (a few chunks read again, a handful of candidates) is a chain of
// memory round trips and wave-wide sums: up to 64 candidates are one wave's, held in registers, with no barrier
// after the list is made.  Many rows run with 512 threads each, so that twice as many are in flight (48 heads x 64 rows of
// 32768 keys, this kernel: 60 us with 1024).  256 would leave long supports half of the chip's waves, since LDS holds four
// rows to a CU (48 heads x 64 rows of 8192 keys, delta = 0, gamma = -1/2, whole call: 908 against 1971 us; 676 with the
// value rows of four keys requested together; 849 with 1024 threads and one value row at a time).
template <typename T, int D, int AM, int NT>
__global__ __launch_bounds__(NT) void decode_solve_kernel(DecodeArgs A) {
  constexpr int kW = NT / 64;
  constexpr int kSlots = NT / D;                   // threads with the same feature share out the support
  __shared__ float2 list[kDecodeListCap];          // (key index bits, z)
  __shared__ float red[2 * 2 * kW];
  __shared__ float wmax[kW], wtop[kW];
  __shared__ int count;
  __shared__ float osum[kSlots * D];
  const Geom& g = A.g;
  const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
  const int row = blockIdx.x, i = row % g.Nq, bh = row / g.Nq, b = bh / g.H, h = bh % g.H;
  const int lim = row_limit(g, i);
  const long long o_idx = (long long)b * g.q_sb + (long long)h * g.q_sh + (long long)i * g.q_sn;
  if (lim == 0) {  // no visible key: an empty sum
    if (tid < D) Elem<T>::store(A.O, o_idx + tid, 0.f);
    if (tid == 0) A.tau[row] = 0.f;
    return;
  }
  float* z = A.scores + (long long)row * A.nks;
  const uint32_t* cmax = A.cmax + (long long)row * A.nchunks;
  const float r = 1.0f / (g.alpha - 1.0f);
  // lower bound of the row maximum from the chunks' rounded maxima
  uint32_t first_words = kCmaxNone;  // the words of chunks 0..63: every wave's own copy
  if (lane < A.nchunks) first_words = cmax[lane];
  float m = cmax_floor(first_words);
  for (int c = 64 + tid; c < A.nchunks; c += NT) m = fmaxf(m, cmax_floor(cmax[c]));
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) m = fmaxf(m, __shfl_xor(m, off));
  if (lane == 0) wmax[wave] = m;
  if (tid == 0) count = 0;
  __syncthreads();
#pragma unroll
  for (int w = 0; w < kW; ++w) m = fmaxf(m, wmax[w]);
  // keys with a non-zero term at the lowest threshold tau_lo = max - 1 (there the maximum's own term is 1,
  // so the sum is >= 1 and the root is >= tau_lo), or a few more: the waves take the chunks in reach in turn
  const float floor_lo = m - 1.0f;
  // body(first key + 4 * lane, in the chunk; chunk; its word) for the chunks whose word is `wanted`, twice 256 keys each
  auto each_chunk = [&](auto wanted, auto body) {
    int turn = 0;
    for (int c0 = 0; c0 < A.nchunks; c0 += 64) {
      const uint32_t word = c0 == 0 ? first_words : (c0 + lane < A.nchunks ? cmax[c0 + lane] : kCmaxNone);
      unsigned long long hot = __ballot(c0 + lane < A.nchunks && wanted(word));
      while (hot != 0ull) {
        const int k = __builtin_ctzll(hot);
        hot &= hot - 1ull;
        if ((turn++ % kW) != wave) continue;
        const uint32_t written = (uint32_t)__builtin_amdgcn_readlane((int)word, k);
#pragma unroll
        for (int v = 0; v < kDecodeChunk / 256; ++v) {
          const int in_chunk = (v * 64 + lane) * 4;
          body((c0 + k) * kDecodeChunk + in_chunk, ((written >> (in_chunk >> 5)) & 1u) != 0u);
        }
      }
    }
  };
  float top = -kInf;  // the largest score itself
  each_chunk([&](uint32_t word) { return (word & 0xffffu) != 0u && cmax_ceil(word) > floor_lo; },
             [&](int j, bool written) {
               if (j >= lim || !written) return;
               const f32x4_t zv = *reinterpret_cast<const f32x4_t*>(z + j);  // nks is a multiple of 4: the word is inside the row
#pragma unroll
               for (int kk = 0; kk < 4; ++kk) {
                 if (j + kk < lim && zv[kk] > floor_lo) {
                   top = fmaxf(top, zv[kk]);
                   const int pos = atomicAdd(&count, 1);
                   if (pos < kDecodeListCap) list[pos] = make_float2(__int_as_float(j + kk), zv[kk]);
                 }
               }
             });
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) top = fmaxf(top, __shfl_xor(top, off));
  if (lane == 0) wtop[wave] = top;
  __syncthreads();
  const int total = count;
#pragma unroll
  for (int w = 0; w < kW; ++w) top = fmaxf(top, wtop[w]);
  // (no candidate at all: the largest score, which is then m exactly, is infinite or so large that one less is the same number)
  float tau = (total > 0 ? top : m) - 1.0f;
  const T* Vh = reinterpret_cast<const T*>(A.V) + (long long)b * g.kv_sb + (long long)h * g.kv_sh;
  auto value = [&](int j, int c) -> float {
    const long long vi = (long long)j * g.kv_sn + c;
    if constexpr (sizeof(T) == 2)
      return __uint_as_float((uint32_t)reinterpret_cast<const uint16_t*>(Vh)[vi] << 16);
    else
      return reinterpret_cast<const float*>(Vh)[vi];
  };
  if (total <= 64) {
    if (wave != 0) return;
    const float2 en = lane < total ? list[lane] : make_float2(0.f, -kInf);
    for (int it = 0; total > 0 && it < 96; ++it) {
      const float x = fmaxf(en.y - tau, 0.f);
      float F = x > 0.f ? pow_r<AM>(x, r) : 0.f, G = x > 0.f ? pow_rm1<AM>(x, r) : 0.f;
#pragma unroll
      for (int off = 32; off >= 1; off >>= 1) {
        F += __shfl_xor(F, off);
        G += __shfl_xor(G, off);
      }
      if (decode_newton(F, G, r, tau)) break;
    }
    if (lane == 0) A.tau[row] = tau;
    const float x = lane < total ? fmaxf(en.y - tau, 0.f) : 0.f;
    const float p = x > 0.f ? pow_r<AM>(x, r) : 0.f;
    unsigned long long sup = __ballot(p > 0.f);
    float acc[D / 64];
#pragma unroll
    for (int t = 0; t < D / 64; ++t) acc[t] = 0.f;
    while (sup != 0ull) {  // four value rows on their way at a time (a row past the last one has weight zero)
      float pe[4], ve[4][D / 64];
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const int k = sup != 0ull ? __builtin_ctzll(sup) : 0;
        pe[u] = sup != 0ull ? __int_as_float(__builtin_amdgcn_readlane(__float_as_int(p), k)) : 0.f;
        const int j = __builtin_amdgcn_readlane(__float_as_int(en.x), k);
        sup &= sup - 1ull;  // (0 stays 0)
#pragma unroll
        for (int t = 0; t < D / 64; ++t) ve[u][t] = value(j, t * 64 + lane);
      }
#pragma unroll
      for (int u = 0; u < 4; ++u)
#pragma unroll
        for (int t = 0; t < D / 64; ++t)
          if (pe[u] > 0.f) acc[t] = fmaf(pe[u], ve[u][t], acc[t]);
    }
#pragma unroll
    for (int t = 0; t < D / 64; ++t) Elem<T>::store(A.O, o_idx + t * 64 + lane, acc[t]);
    return;
  }
  // tau, then the thread's share of O_i = sum_j p_ij v_j over n items; B items' scores and value rows are requested at a
  // time, the sum runs in their order
  const int slot = tid / D, c = tid % D;
  float acc = 0.f;
  auto solve = [&](auto key_of, auto score_of, int n, auto b_tag) {
    constexpr int B = decltype(b_tag)::value;
    for (int it = 0; it < 96; ++it) {
      float F = 0.f, G = 0.f;
      for (int e = tid; e < n; e += NT) {
        const float x = score_of(e) - tau;
        if (x > 0.f) {
          F += pow_r<AM>(x, r);
          G += pow_rm1<AM>(x, r);
        }
      }
      const float2 s = decode_block_sum<NT>(F, G, red, it & 1);
      if (decode_newton(s.x, s.y, r, tau)) break;
    }
    for (int e0 = slot; e0 < n; e0 += B * kSlots) {
      float x[B], v[B];
#pragma unroll
      for (int u = 0; u < B; ++u) x[u] = e0 + u * kSlots < n ? score_of(e0 + u * kSlots) - tau : 0.f;
#pragma unroll
      for (int u = 0; u < B; ++u) v[u] = x[u] > 0.f ? value(key_of(e0 + u * kSlots), c) : 0.f;
#pragma unroll
      for (int u = 0; u < B; ++u)
        if (x[u] > 0.f) acc = fmaf(pow_r<AM>(x[u], r), v[u], acc);
    }
  };
  if (total <= kDecodeListCap) {
    solve([&](int e) { return __float_as_int(list[e].x); }, [&](int e) { return list[e].y; }, total, std::integral_constant<int, 1>());
  } else {
    // the row itself is read again and again: the scores that were not written become -inf once and for all
    each_chunk([&](uint32_t word) { return (word & 0xffffu) != 0xffffu; },
               [&](int j, bool written) {
                 if (j < A.nks && !written) *reinterpret_cast<f32x4_t*>(z + j) = f32x4_t{-kInf, -kInf, -kInf, -kInf};
               });
    __syncthreads();
    solve([](int e) { return e; }, [&](int e) { return z[e]; }, lim, std::integral_constant<int, 4>());
  }
  if (tid == 0) A.tau[row] = tau;
  osum[slot * D + c] = acc;
  __syncthreads();
  if (tid < D) {
    float o = 0.f;
#pragma unroll
    for (int s = 0; s < kSlots; ++s) o += osum[s * D + tid];
    Elem<T>::store(A.O, o_idx + tid, o);
  }
}

}  // namespace entmax
