// Forward path for rows whose support is small (the regime the paper's
// ASEntmax workloads live in: a handful of non-zero probabilities per row).
//
// alpha-entmax gives exact zeros below the threshold (Sec. 2.2, App. A), and the
// threshold is bounded below by any sub-problem: solving eq. (entmax) on a
// subset S of the row's scores gives tau_S <= tau, because dropping terms can
// only lower f(tau) = sum_j [(alpha-1) s_j - tau]_+^r - 1.  So
//   fwd_lists_kernel (matrix cores, K tiles through LDS, one sweep)
//     1. a sweep over the scores that keeps the row maximum and each lane's (half row's) largest groups of eight keys:
//        tau_lb = max(left end of the bracket of App. A eq. (bounds),
//                     solution of the sub-problem of those groups' largest scores) <= tau;
//     2. the scores of the keys of the groups above tau_lb once more, from memory: every key with (alpha-1) s_ij > tau_lb goes on the
//        row's candidate list (key index + raw score).  Every key of the
//        support is on that list; nothing else of the row can matter.  Rows with more such groups than were kept are
//        looked through on their own; where a block has many of them, or many groups, it is swept a second time instead.
//   fwd_finish_kernel (no matrix work, one lane pair per row)
//     3. the threshold by the same safeguarded steps as the tiled kernel
//        (closed-form local-model root for alpha 1.5 / 2, Halley / Newton
//        otherwise), summing over the list instead of over key tiles;
//     4. O_i = sum over the list of p_ij v_j, gathering the few value rows; for the
//        backward, the entries with p_ij > 0 are written out as the row's support list.
// A workgroup that meets a row with more candidates than a list holds raises
// its flag and leaves the whole block to the tiled kernel (fwd.hip.h), which
// handles any density.
// Also here: what the other list kernels share (bwd_sparse.hip.h, decode.hip.h): the
// slot-major list layout, the collect sweep, row gather helpers.
#pragma once
#include "fwd.hip.h"
#include "transpose.hip.h"

namespace entmax {

// Row lists (candidates, supports, per-entry records) are stored per wave of 32 rows x 2 halves with
// entry s of all 64 lanes together: short lists then touch only the first few 512-byte groups of a
// wave's region instead of one cache line per half row.  Wave w = ((bh * nqb + qb) * 4 + wave in block);
// entry (lane, s) sits at list_entry<CAP>(w, lane) + s * kListStride.
template <int CAP>
__device__ __forceinline__ long long list_entry(int bh, int nqb, int qb, int wave, int lane) {
  return (((long long)bh * nqb + qb) * kWaves + wave) * CAP * kListStride + lane;
}


struct FwdSparseArgs {
  Geom g;
  const void* Q;
  const void* K;
  const void* V;
  void* O;
  float* tau;
  uint2* cand;      // [B*H*nqb*4 waves][kCandCap][64 lanes] (key index, raw dot product bits), see list_entry()
  uint2* list;      // NULL, or the pool of the `saved` buffer the rows' supports are packed into for the backward:
                    // every 32-row group takes one contiguous piece (lane after lane, entry after entry)
  char* pool_cursor;       // with list: the pool's parts each have a 64-bit cursor (entries handed out so far, zeroed
                           // by the list kernel), kSavedCursorStride bytes apart
  int pool_shift;          // with list: the pool is cut into 1 << pool_shift parts
  long long pool_part_cap; // with list: entries a part holds
  int* slcnt;       // with list: [B*H*Nq][2] per half row: (place of its first entry in the pool) << 5 | entries
  int* bwd_flag;    // with list: [B*H*nqb] not 0: the backward cannot take its list path for this block
                    // (kBlockListsUnused, kBlockNoLists)
  int* kcount;      // with list: [B*H*Nk] support entries naming each key (zeroed by the list kernel, counted by
                    // the finish kernel): the sizes of the backward's key-major segments
  void* cells;      // sweep scratch: one CellBuf<kCandCap> per workgroup of the list sweep's grid
  int* lcnt;        // [B*H*Nq][2] list lengths
  float2* bounds;   // [B*H*Nq] (tau_lb, right end of the bracket)
  int* dense_flag;  // [B*H*nqb] above zero: block left to the tiled kernel (kFlagDense, kFlagWithBounds), else lists
                    // were made: minus what the block asks of the pool (pool_want()).  Behind them: how many
                    // are left to the tiled kernel (zeroed by the list kernel, counted by the finish kernel), then the
                    // first kSplitMaxBlocks of these blocks' numbers
  unsigned long long* stats;
  int nqb;
  int force_long;      // run the long-sequence kernels whatever the sizes (params.path = 2: test aid)
  int unpaired;        // fwd_lists_kernel: one query block per workgroup (see fwd_lists_unpaired())
  TransposeRide ride;  // V^T copies for the tiled kernel, as extra workgroups of the finish launch
};

// A cell is a group of four consecutive accumulator registers of a lane (keys j, j+1, j+2, j+3 of
// one row).  During a sweep a lane appends whole cells
// -- all their raw scores and the first key index -- to a private strip of scratch memory whenever the
// cell maximum passes the cutoff: one short divergent region per cell instead of one per score.  After
// the sweep each lane walks its own cells and writes the scores above the cutoff to its list.
// The first LS cells of a thread stay in LDS (the common case: a row has a handful of candidates), the others go
// to a strip of global scratch.  Addresses are formed where they are used: the struct holds two registers.
template <int CAP, int LS>
struct CellBuf {
  static_assert(kCellGroups == 1, "a cell is one group of four accumulator registers");
  // cell s of the 256 threads of a workgroup together (s-major), for the same reason as the row lists:
  //   LDS:    scores of cell s at lds + (s * kThreads + tid) * 16, its first key at lds + LS * kThreads * 16 + (s * kThreads + tid) * 4
  //   global: the same with CAP in place of LS, in the workgroup's strip
  char* lds;
  char* strip;  // workgroup-uniform
  int tid;
  int in_lds;  // cells of a thread that go to LDS (LS, or 0)
  static constexpr size_t kBytesPerWorkgroup = cell_bytes_per_workgroup(CAP);
  static constexpr int kLdsBytes = LS * kThreads * 20;
  __device__ __forceinline__ void init(void* base, char* lds_, int tid_, int strip_no = blockIdx.x) {
    strip = reinterpret_cast<char*>(base) + (size_t)strip_no * kBytesPerWorkgroup;
    lds = lds_;
    tid = tid_;
    in_lds = LS;
  }
  // n: cells this thread stored before.  A strip that is full keeps overwriting its last cell (the caller
  // then discards the lists).
  __device__ __forceinline__ void store(int n, const f32x4_t& v, int key) {
    if (LS > 0 && n < in_lds) {
      const int e = n * kThreads + tid;
      *reinterpret_cast<f32x4_t*>(lds + e * 16) = v;
      *reinterpret_cast<int*>(lds + LS * kThreads * 16 + e * 4) = key;
    } else {
      const int e = min(n, CAP - 1) * kThreads + tid;
      *reinterpret_cast<f32x4_t*>(strip + (size_t)e * 16) = v;
      *reinterpret_cast<int*>(strip + (size_t)CAP * kThreads * 16 + (size_t)e * 4) = key;
    }
  }
  __device__ __forceinline__ void load(int n, f32x4_t& v, int& key) const {
    if (LS > 0 && n < in_lds) {
      const int e = n * kThreads + tid;
      v = *reinterpret_cast<const f32x4_t*>(lds + e * 16);
      key = *reinterpret_cast<const int*>(lds + LS * kThreads * 16 + e * 4);
    } else {
      const int e = n * kThreads + tid;
      v = *reinterpret_cast<const f32x4_t*>(strip + (size_t)e * 16);
      key = *reinterpret_cast<const int*>(strip + (size_t)CAP * kThreads * 16 + (size_t)e * 4);
    }
  }
};

// Scores acc of the 32-key block at key j0 (masked where the row does not see the key): appends the cells above the cutoff.
template <typename C, typename CB>
__device__ __forceinline__ void append_cells(const C& q, const f32x16_t& acc, int j0, float cut, CB& cb, int& ncell,
                                             unsigned& n_cand_tiles) {
  // maxima of the four 4-key groups of the lane, then of the block
  float gm[4];
#pragma unroll
  for (int gq = 0; gq < 4; ++gq) gm[gq] = fmaxf(fmaxf(acc[4 * gq], acc[4 * gq + 1]), fmaxf(acc[4 * gq + 2], acc[4 * gq + 3]));
  const float lm = fmaxf(fmaxf(gm[0], gm[1]), fmaxf(gm[2], gm[3]));
  // masked entries are -inf and never exceed the cutoff
  if (__ballot(lm > cut) == 0ull) return;
  ++n_cand_tiles;
#pragma unroll
  for (int cl = 0; cl < 4; ++cl) {
    if (gm[cl] > cut) {
      cb.store(ncell, f32x4_t{acc[4 * cl], acc[4 * cl + 1], acc[4 * cl + 2], acc[4 * cl + 3]}, j0 + q.key_of(4 * cl));
      ++ncell;
    }
  }
}

// keys of the block at j0 that the lane's row does not see
template <typename C>
__device__ __forceinline__ void mask_block(const C& q, f32x16_t& acc, int j0) {
  const int rel = q.lim - j0;
#pragma unroll
  for (int e = 0; e < 16; ++e) acc[e] = (q.key_of(e) < rel) ? acc[e] : -kInf;
}

// A cell holds at most four candidates, so there are at least as many candidates as cells.  One pass: the scores
// above the cutoff go to the list.  Returns how many there are; more than CAP: the block's lists are discarded.
// Four cells are read at a time: one after the other they are a chain of memory round trips (forward, 12 heads: B 4, n 4096, alpha 1.25
// 406 -> 399 us, no scale 660 -> 645; 8 heads, n 1100, alpha 1.7, no scale 79.6 -> 77.6).
template <int CAP, typename CB>
__device__ __forceinline__ int cells_to_list(const CB& cb, int ncell, float cut, uint2* mylist, int& cnt) {
  int total = 0;
  constexpr int P = 4;  // cells under way at a time
  for (int k = 0; k < ncell; k += P) {
    f32x4_t dv[P];
    int jc[P];
#pragma unroll
    for (int u = 0; u < P; ++u)
      if (k + u < ncell) cb.load(k + u, dv[u], jc[u]);
#pragma unroll
    for (int u = 0; u < P; ++u) {
      if (k + u >= ncell) break;
#pragma unroll
      for (int rr = 0; rr < 4; ++rr) {
        if (dv[u][rr] > cut) {
          if (cnt < CAP) {
            mylist[cnt * kListStride] = make_uint2((unsigned)(jc[u] + rr), __float_as_uint(dv[u][rr]));
            ++cnt;
          }
          ++total;
        }
      }
    }
  }
  return total;
}

// candidates are the keys with a * dot > thr: in raw units, dot > cut.  Rounding may move a key that
// sits on the threshold (probability ~ 0) in or out of the list; the consumers recompute its value.
// Scale 0 (a = 0): every visible key ties; they all qualify iff thr < 0.
__device__ __forceinline__ float raw_cut(float a, bool live, float thr) {
  return !live ? kInf : (a > 0.f ? thr / a : (thr < 0.f ? -3.0e38f : kInf));
}

// What a block asks of the `saved` pool, before its supports are known: a half row's support is part of its candidate
// list, and more than kBwdCap entries of one half row send the block to the backward's tiled kernels.  So: the sum of
// min(candidates, kBwdCap) in the low 16 bits (256 half rows: at most 4096), and above them how many of the block's four
// row groups hold a half row with more candidates than that -- where none does, the block's lists are sure to be used.
// word: LDS, zero before; complete after the workgroup's next barrier.
__device__ __forceinline__ void pool_want(int* word, int cnt, int lane) {
  const int c = min(cnt, kBwdCap);
  int sum = 0;
#pragma unroll
  for (int k = 0; k < 5; ++k) sum += (int)__popcll(__ballot(((c >> k) & 1) != 0)) << k;
  const int longer = __ballot(cnt > kBwdCap) != 0ull ? 1 << 16 : 0;
  if (lane == 0) atomicAdd(word, sum | longer);
}
static_assert(kBwdCap < 32 && kThreads * kBwdCap < (1 << 16), "five bits a half row, 16 a block");

// One sweep over the visible key tiles of the block: every key whose raw score exceeds the lane's cut ends up in its
// list, behind the cnt entries that are there.  Returns false (workgroup-uniform) if
// some list overflowed; the sweep is abandoned early in that case.  ovf: three ints of LDS;
// lds_cells: CellBuf<CAP, LS>::kLdsBytes bytes of LDS.  wave_on (wave-uniform): false: no lane of this wave looks for
// anything, and it only helps to bring the tiles.  With the forward's lists (CAP = kCandCap), ovf[3] is a word for pool_want().
template <typename C, typename T, int D, int CAP, int LS, bool RING = false>
__device__ __forceinline__ bool collect_sweep(const C& q, const Geom& g, const void* K, char* tiles, int* ovf, char* lds_cells,
                                              float cut, void* cells, uint2* mylist, int& cnt, unsigned& n_qk,
                                              unsigned& n_cand_tiles, bool wave_on = true, int strip_no = -1) {
  constexpr int KT = C::KT, NSB = C::NSB;
  if (q.tid < 3) ovf[q.tid] = 0;
  CellBuf<CAP, LS> cb;
  cb.init(cells, lds_cells, q.tid, strip_no < 0 ? (int)blockIdx.x : strip_no);  // (which of the scratch strips is this workgroup's)
  if constexpr (RING && LS > 0) {  // (the cells' LDS is the ring's third buffer)
    int first = 0;
    if constexpr (C::BIAS) first = q.kt_first;
    if (q.ntiles - first > 2) cb.in_lds = 0;
  }
  int ncell = 0;
  Slot slots[1];
  slots[0].base = reinterpret_cast<const char*>(reinterpret_cast<const T*>(K) + (long long)q.b * g.kv_sb +
                                                (long long)q.h * g.kv_sh);
  slots[0].row_bytes = g.kv_sn * (long long)sizeof(T);
  auto body = [&](int kt, const char* tl) {
    if (!wave_on || !q.tile_in_wave_window(kt)) return;
    const bool interior = (kt + 1) * KT <= q.wave_lim_min;
    const uint32_t act = interior ? ((1u << NSB) - 1u) : q.visible_bits(kt);
    if (act == 0u) return;
    f32x16_t acc[NSB];
    if (interior) {
      q.scores_all(tl, acc, kt);
    } else {
#pragma unroll
      for (int sb = 0; sb < NSB; ++sb)
        if (act & (1u << sb)) acc[sb] = q.scores(tl, sb, kt);
    }
#pragma unroll
    for (int sb = 0; sb < NSB; ++sb) {
      if (!(act & (1u << sb))) continue;
      int j0 = kt * KT + sb * 32;
      ++n_qk;
      if (j0 + 32 > q.wave_lim_min) mask_block(q, acc[sb], j0);
      append_cells(q, acc[sb], j0, cut, cb, ncell, n_cand_tiles);
    }
    // once per tile: a strip that overflowed (its last cell was overwritten: the lists are discarded)
    if (__ballot(ncell > CAP) != 0ull && q.lane == 0) ovf[kt & 1] = 1;
  };
  // flags of the previous tile's parity were final before the barrier that ended that tile
  auto leave = [&](int kt) { return kt > 0 && ovf[(kt - 1) & 1] != 0; };
  if constexpr (RING) {
    TileRing<C, T, D> ring;
    int first = 0;
    if constexpr (C::BIAS) first = q.kt_first;
    ring.start(tiles, slots[0], first, q.ntiles, g.Nk);
    while (ring.kt < q.ntiles && !leave(ring.kt)) ring.step([&](const char* tl) { body(ring.kt, tl); });
    ring.abandon();
  } else {
    sweep_tiles<C, T, D, 1, 0, ListCfg<T, D>::kDepth>(tiles, slots, q.ntiles, g.Nk, q.tid, [&](int kt) { return q.tile_in_window(kt); },
                                                      body, leave);
  }
  // the sweep ended on a barrier: both flags are final
  bool fits = (ovf[0] | ovf[1]) == 0;
  if (fits) {
    const int total = cells_to_list<CAP>(cb, ncell, cut, mylist, cnt);
    if (total > CAP) ovf[2] = 1;
    if constexpr (CAP == kCandCap) pool_want(ovf + 3, cnt, q.lane);
    __syncthreads();
    fits = ovf[2] == 0;
  }
  return fits;
}

// The sweep's memory of where a lane's large scores are: its kTopGroups largest groups by the lane's largest score of
// each, in descending order.  A group is G (8 or 16) of the lane's 16 accumulator registers of a 32-key block; an entry is that score with
// the group's number in place of its lowest mantissa bits, so that one v_med3 per place keeps the order (t1 >= t2: the middle
// one of t1, t2, x is the new t2).  The entries give a lower bound of the threshold from up to sixteen scores (top_groups_bound()), and
// those above it name every key that can be in the support: only these keys' scores are formed again (rescore_groups()),
// and the sweep over the scores need not be repeated.
constexpr int kTopGroups = 12;
// Rows of strong scales need fewer places: a wave all of whose rows have (alpha-1) |scale| of kFewPlacesScale or more keeps this
// many while it goes through the tiles that every row sees whole.  (Normal scores, alpha 1.5, n 1024 to 32768: of the lanes whose
// (alpha-1) |scale| is 2.3 fewer than 1 in 1000 need more than eight, at 1.2 one to three in 100, of which 1 in 500 more than twelve.  Places cost
// two vector instructions a block and each: with eight for all n 4096 101 us, n 32768 1060, with twelve for all the sweep 6 us longer.)
constexpr int kFewPlaces = 8;
constexpr float kFewPlacesScale = 3.0f;
template <int G>
struct GroupNumbers {  // how the numbers of a head's groups are packed
  static constexpr int kPerBlock = 16 / G;  // groups of a lane in a 32-key block
  uint32_t keep;       // the score's bits that stay
  float eps;           // a score differs from its entry by less than eps |entry|
  __device__ __forceinline__ explicit GroupNumbers(int Nk) {
    const int bits = 32 - __builtin_clz((unsigned)(((Nk - 1) >> 5) * kPerBlock + kPerBlock - 1) | 1u);
    keep = ~((1u << bits) - 1u);
    asm volatile("" : "+v"(keep));  // (in a vector register: an instruction takes one scalar operand, the group's number)
    eps = __uint_as_float((uint32_t)(127 + bits - 22) << 23);
  }
  __device__ __forceinline__ float upper(float t) const { return fmaf(fabsf(t), eps, t); }  // (both increasing in t)
  __device__ __forceinline__ float lower(float t) const { return fmaf(-fabsf(t), eps, t); }
};
template <int G>
struct TopGroups {
  using Numbers = GroupNumbers<G>;
  float t[kTopGroups];
  __device__ __forceinline__ void init() {
#pragma unroll
    for (int k = 0; k < kTopGroups; ++k) t[k] = __uint_as_float(0xff700000u);  // below every entry (-3.19e38)
  }
  __device__ __forceinline__ void take_one(float m, const Numbers& gn, int number) {
    const float x = __uint_as_float((__float_as_uint(m) & gn.keep) | (uint32_t)number);
#pragma unroll
    for (int k = kTopGroups - 1; k > 0; --k) t[k] = __builtin_amdgcn_fmed3f(t[k - 1], t[k], x);
    t[0] = fmaxf(t[0], x);
  }
  // the lane's 16 scores of block jb; returns the largest.  No entry is below `floor`: kFloor keeps the bits of a masked
  // group's -inf from becoming a NaN; with kNothing, which is below what init() left, scores of -inf leave no entry.  (An infinite
  // score may leave a NaN; its row has an infinite bound, and no key passes it.)
  static constexpr float kFloor = -3.0e38f, kNothing = -3.4e38f;
  __device__ __forceinline__ float take(const f32x16_t& acc, const Numbers& gn, int jb, float floor = kFloor) {
    constexpr int P = GroupNumbers<G>::kPerBlock;
    float m[P];
#pragma unroll
    for (int u = 0; u < P; ++u) {
      m[u] = fmaxf(fmaxf(acc[G * u], acc[G * u + 1]), floor);
#pragma unroll
      for (int e = 2; e < G; e += 2) m[u] = fmaxf(fmaxf(m[u], acc[G * u + e]), acc[G * u + e + 1]);
      take_one(m[u], gn, P * jb + u);
    }
    return P == 1 ? m[0] : fmaxf(m[0], m[P - 1]);
  }
  // the same in four parts of about equally many instructions, to be issued between matrix instructions; m, x: the caller's, kept
  // from part to part
  template <int PART, int K>
  __device__ __forceinline__ void take_part(const f32x16_t& acc, const Numbers& gn, int jb, float floor, float (&m)[16 / G],
                                            float (&x)[16 / G], float& most) {
    constexpr int P = GroupNumbers<G>::kPerBlock, N = P * K;
    if constexpr (PART == 0) {
#pragma unroll
      for (int u = 0; u < P; ++u) m[u] = fmaxf(fmaxf(acc[G * u], acc[G * u + 1]), floor);
#pragma unroll
      for (int e = 2; e < G; e += 2)
#pragma unroll
        for (int u = 0; u < P; ++u) m[u] = fmaxf(fmaxf(m[u], acc[G * u + e]), acc[G * u + e + 1]);
    } else {
      if constexpr (PART == 1) {
#pragma unroll
        for (int u = 0; u < P; ++u) {
          int number = P * jb + u;
          asm volatile("" : "+s"(number));  // (one instruction for both steps)
          x[u] = __uint_as_float((__float_as_uint(m[u]) & gn.keep) | (uint32_t)number);
        }
        most = P == 1 ? fmaxf(most, m[0]) : fmaxf(fmaxf(most, m[0]), m[P - 1]);
      }
#pragma unroll
      for (int op = (PART - 1) * N / 3; op < PART * N / 3; ++op) {
        const int u = op / K, k = K - 1 - op % K;
        t[k] = k > 0 ? __builtin_amdgcn_fmed3f(t[k > 0 ? k - 1 : 0], t[k], x[u]) : fmaxf(t[0], x[u]);
      }
    }
  }
  // how many of the entries may name a candidate
  __device__ __forceinline__ int above(float cut, const Numbers& gn) const {
    int n = 0;
#pragma unroll
    for (int k = 0; k < kTopGroups; ++k) n += (t[k] > -3.1e38f && gn.upper(t[k]) > cut) ? 1 : 0;
    return n;
  }
  // the row's second largest group maximum (a little low): a second, distinct score; below -2.9e38: there is none
  __device__ __forceinline__ float runner_up(const Numbers& gn) const {
    const float p0 = __shfl_xor(t[0], 32), p1 = __shfl_xor(t[1], 32);
    return gn.lower(fmaxf(fminf(t[0], p0), fmaxf(t[1], p1)));
  }
};

// Sum over the eight lanes of an octet of eight values each: lane c of the octet gets the sum of value kMap(c) (see
// octet_value()).  Each step sends half of the values to the partner and keeps the other half.
template <int CTRL>
__device__ __forceinline__ float dpp_move(float v) {
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, 0xf, 0xf, true));
}
__device__ __forceinline__ float octet_scatter_sum(const float (&s)[8], int c) {
  const bool b2 = (c & 4) != 0, b1 = (c & 2) != 0, b0 = (c & 1) != 0;
  float u[4], v[2];
#pragma unroll
  for (int k = 0; k < 4; ++k)  // partner 7 - c (row_half_mirror): lanes 4 to 7 keep values 4 to 7
    u[k] = (b2 ? s[k + 4] : s[k]) + dpp_move<0x141>(b2 ? s[k] : s[k + 4]);
#pragma unroll
  for (int k = 0; k < 2; ++k)  // partner c ^ 2 (quad_perm 2 3 0 1)
    v[k] = (b1 ? u[k + 2] : u[k]) + dpp_move<0x4e>(b1 ? u[k] : u[k + 2]);
  return (b0 ? v[1] : v[0]) + dpp_move<0xb1>(b0 ? v[0] : v[1]);  // partner c ^ 1 (quad_perm 1 0 3 2)
}

typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
// acc + a.lo * b.lo + a.hi * b.hi for two packed bf16 pairs, in fp32
__device__ __forceinline__ float dot2_bf16(uint32_t a, uint32_t b, float acc) {
  return __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2_t, a), __builtin_bit_cast(bf16x2_t, b), acc, false);
}

// Scores of the keys of groups, from memory.  Eight lanes (an octet) take a group, each lane a 16-byte word of every 128 bytes of
// a key row, so that a load instruction brings eight whole rows (D 64, bf16).
template <typename C, typename T, int D, int G>
struct OctetScores {
  static constexpr int W = D * (int)sizeof(T) / 128;  // 16-byte words of a row per lane
  static constexpr int KB = W <= 2 ? 8 : 4;           // keys whose words are requested together
  static constexpr int P = GroupNumbers<G>::kPerBlock;
  struct Row {  // the octet's row
    int pos, lim;
    float cut, w;
    bool negated;
    u32x4_t qw[W];
  };
  const Geom& g;
  const char *Kbh, *Qbh;
  uint32_t krow_bytes;
  int c, q0;  // lane of the octet; first row of the wave
  __device__ __forceinline__ OctetScores(const C& q, const Geom& g_, const void* Q, const void* K) : g(g_) {
    c = q.lane & 7;
    q0 = q.q0;
    Kbh = reinterpret_cast<const char*>(reinterpret_cast<const T*>(K) + (long long)q.b * g.kv_sb + (long long)q.h * g.kv_sh) + 16 * c;
    Qbh = reinterpret_cast<const char*>(reinterpret_cast<const T*>(Q) + (long long)q.b * g.q_sb + (long long)q.h * g.q_sh) + 16 * c;
    krow_bytes = (uint32_t)(g.kv_sn * (long long)sizeof(T));
  }
  // id: the lane of the wave whose keys are looked at; all lanes of the wave call this together
  __device__ __forceinline__ Row row(const C& q, float wave_cut, int id) const {
    float w = 0.f;
    if constexpr (C::BIAS) w = __shfl(q.w, id);
    return row_of(q0 + (id & 31), __shfl(wave_cut, id), __shfl(q.c, id) < 0.f, w);
  }
  __device__ __forceinline__ Row row_of(int i, float cut, bool negated, float w) const {
    Row r;
    r.pos = i + (g.Nk - g.Nq);
    r.lim = g.causal ? min(r.pos + 1, g.Nk) : g.Nk;
    const char* qrow = Qbh + (long long)i * (g.q_sn * (long long)sizeof(T));
#pragma unroll
    for (int k = 0; k < W; ++k) r.qw[k] = *reinterpret_cast<const u32x4_t*>(qrow + 128 * k);
    r.cut = cut;
    r.negated = negated;
    r.w = w;
    return r;
  }
  // first key of group `number` of a lane of half hh; register r of the group: key 8 (r / 4) + r % 4 behind it
  static __device__ __forceinline__ int first_key(int number, int hh) { return (number / P) * 32 + (number % P) * 16 + 4 * hh; }
  __device__ __forceinline__ int key(int j0, int r0) const { return j0 + 8 * ((r0 + c) >> 2) + (c & 3); }
  // scores of registers r0 .. r0 + 7 of N groups at keys j0[]: lane c gets that of register r0 + c
  template <int N>
  __device__ __forceinline__ void eight(const Row (&row)[N], const int (&j0)[N], int r0, float (&d)[N]) const {
    float part[N][8];
#pragma unroll
    for (int rb = 0; rb < 8; rb += KB) {
      u32x4_t kw[N][KB][W];
#pragma unroll
      for (int n = 0; n < N; ++n)
#pragma unroll
        for (int u = 0; u < KB; ++u) {
          const int r = r0 + rb + u;
          const int j = min(j0[n] + 8 * (r >> 2) + (r & 3), g.Nk - 1);  // (rows beyond the tensor: masked by lim)
          const char* krow = Kbh + (unsigned long long)(uint32_t)j * krow_bytes;
#pragma unroll
          for (int k = 0; k < W; ++k) kw[n][u][k] = *reinterpret_cast<const u32x4_t*>(krow + 128 * k);
        }
      __builtin_amdgcn_sched_barrier(0);  // (all of them requested before the first is used)
#pragma unroll
      for (int n = 0; n < N; ++n)
#pragma unroll
        for (int u = 0; u < KB; ++u) {
          float s = 0.f;
#pragma unroll
          for (int k = 0; k < W; ++k) {
#pragma unroll
            for (int e = 0; e < 4; ++e) {
              if constexpr (sizeof(T) == 2)
                s = dot2_bf16(kw[n][u][k][e], row[n].qw[k][e], s);
              else
                s = fmaf(__uint_as_float(kw[n][u][k][e]), __uint_as_float(row[n].qw[k][e]), s);
            }
          }
          part[n][rb + u] = s;
        }
    }
#pragma unroll
    for (int n = 0; n < N; ++n) {
      d[n] = octet_scatter_sum(part[n], c);
      if (row[n].negated) d[n] = -d[n];
      if constexpr (C::BIAS) d[n] = fmaf(row[n].w, (float)bias_dist(row[n].pos, key(j0[n], r0)), d[n]);
    }
  }
};

constexpr int kRescoreWords = 64 * (kTopGroups + 1);  // of LDS, per wave, for rescore_groups()
// A word of rescore_groups(): the lane (6 bits), the group's number (Nk <= 2^22: at most 18 bits), and which of the seven words before it,
// as far as they are in its own eight, are the same lane's (bit o: word o of the eight).
constexpr int kNumberBits = 18, kBeforeShift = 6 + kNumberBits;

// The keys of the groups that the lanes' first `ne` entries name: their scores, and those above the row's cut go on the
// lists.  The octets of the wave take the groups in turn, two at a time (D 64, bf16) so that sixteen groups are under way.
// lds: kRescoreWords words of the wave's own.  wave_list: the wave's lists, entry s of lane l at s * kListStride + l.  Returns
// false if the lane's list is too short.
template <typename C, typename T, int D, int G>
__device__ __forceinline__ bool rescore_groups(const C& q, const Geom& g, const void* Q, const void* K, const TopGroups<G>& top,
                                               const GroupNumbers<G>& gn, float cut, int ne, int* lds, uint2* wave_list, int& cnt) {
  using O = OctetScores<C, T, D, G>;
  constexpr int N = O::W == 1 ? 2 : 1;  // groups an octet has under way
  int* counts = lds;
  int* slots = lds + 64;
  const int oct = q.lane >> 3;
  const O o(q, g, Q, K);
  const int c = o.c;
  auto lanes_below = [](unsigned long long m) {
    return (int)__builtin_amdgcn_mbcnt_hi((unsigned)(m >> 32), __builtin_amdgcn_mbcnt_lo((unsigned)m, 0u));
  };
  counts[q.lane] = 0;
  int n = 0, last = -8;
  uint32_t earlier = 0u;
#pragma unroll
  for (int k = 0; k < kTopGroups; ++k) {
    const unsigned long long takers = __ballot(k < ne);
    if (k < ne) {
      const int at = n + lanes_below(takers);
      earlier = (at >> 3) == (last >> 3) ? earlier | 1u << (last & 7) : 0u;
      last = at;
      slots[at] = (int)(earlier << kBeforeShift | (__float_as_uint(top.t[k]) & ~gn.keep) << 6) | q.lane;
    }
    n += (int)__popcll(takers);
  }
  __builtin_amdgcn_wave_barrier();
#pragma unroll 1
  for (int s0 = 0; s0 < n; s0 += 8 * N) {
    int id[N], j0[N];
    uint32_t same[N];  // the octets before this one that have a group of its lane
    typename O::Row row[N];
#pragma unroll
    for (int u = 0; u < N; ++u) {
      const uint32_t slot = (uint32_t)slots[min(s0 + 8 * u + oct, n - 1)];
      id[u] = (int)(slot & 63u);
      j0[u] = O::first_key((int)((slot >> 6) & ((1u << kNumberBits) - 1u)), id[u] >> 5);
      same[u] = slot >> kBeforeShift;
      row[u] = o.row(q, cut, id[u]);
      if (s0 + 8 * u + oct >= n) row[u].lim = 0;
    }
#pragma unroll
    for (int r0 = 0; r0 < G; r0 += 8) {
      float d[N];
      o.eight(row, j0, r0, d);
#pragma unroll
      for (int u = 0; u < N; ++u) {
        const int j = o.key(j0[u], r0);
        const bool pass = j < row[u].lim && d[u] > row[u].cut;
        const unsigned long long all = __ballot(pass);
        const unsigned mine = (unsigned)(all >> (8 * oct)) & 0xffu;
        // The octet's place in its list: behind what came in earlier turns and in this one from octets before it.  (The order in which the
        // hardware adds for the lanes of one instruction is not relied on.)
        int at = counts[id[u]] + (int)__popc(mine & ((1u << c) - 1u));
        __builtin_amdgcn_wave_barrier();
        if (c == 0) atomicAdd(counts + id[u], (int)__popc(mine));
        __builtin_amdgcn_wave_barrier();
        if (__ballot(same[u] != 0u) != 0ull) {
#pragma unroll
          for (int k = 0; k < 7; ++k) at += ((same[u] >> k) & 1u) != 0u ? (int)__popc((unsigned)(all >> (8 * k)) & 0xffu) : 0;
        }
        if (pass && at < kCandCap) wave_list[at * kListStride + id[u]] = make_uint2((unsigned)j, __float_as_uint(d[u]));
      }
    }
  }
  __builtin_amdgcn_wave_barrier();
  const int total = counts[q.lane];
  cnt = min(total, kCandCap);
  return total <= kCandCap;
}

// Lower bound of the threshold from the two-element sub-problem {y1 >= y2} (y = (alpha-1) s) and the left
// end y1 - 1 of the bracket of App. A eq. (bounds).  alpha 1.5 and 2: closed forms.  Other alpha: Newton steps
// on f(t) = (y1-t)^r + [y2-t]_+^r - 1 from t = y1 - 1, where f >= 0: f is convex and decreasing, so the
// iterates rise towards the root and stay on its left -- each of them is a valid bound.
template <int AM>
__device__ __forceinline__ float two_key_bound(float y1, float y2, float r) {
  float lo = y1 - 1.0f;
  const float dlt = y1 - y2;
  if (!(dlt < 1.0f)) return lo;  // y2 is zero already at the left end (also y2 = -inf)
  if (AM == 2) return fmaxf(lo, 0.5f * (y1 + y2 - 1.0f));
  float t = lo;
  if (AM == 1) {
    // closed form; the hardware square root is good to an ulp, which the step back below covers
    t = 0.5f * (y1 + y2) - __builtin_amdgcn_sqrtf(0.5f * (1.0f - 0.5f * dlt * dlt));
    return fmaxf(lo, t - 4e-6f * fmaxf(1.0f, fabsf(t)));
  }
#pragma unroll
  for (int it = 0; it < 4; ++it) {
    const float x1 = y1 - t, x2 = fmaxf(y2 - t, 0.f);
    const float f = pow_r<AM>(x1, r) + pow_r<AM>(x2, r) - 1.0f;
    const float fp = r * (pow_rm1<AM>(x1, r) + pow_rm1<AM>(x2, r));
    t += fmaxf(f, 0.f) / fp;  // fp >= r x1^(r-1) > 0 while t < y1
  }
  // rounding may carry the last iterate a few ulps past the root: step back by more than that
  return fmaxf(lo, t - 4e-6f * fmaxf(1.0f, fabsf(t)));
}

// The same from the up to 2 kTopGroups scores of the row that its two lanes' top groups name (distinct keys, each a little
// low), starting at the bound lo: Newton steps from the left, as above.  A row of many close scores has far fewer keys above
// this bound than above the two-key one.
template <int AM, int G>
__device__ __forceinline__ float top_groups_bound(const TopGroups<G>& top, const GroupNumbers<G>& gn, float a, float lo, float r) {
  float v[kTopGroups];
#pragma unroll
  for (int k = 0; k < kTopGroups; ++k) v[k] = a * gn.lower(top.t[k]);
  float t = lo;
#pragma unroll 1
  for (int it = 0; it < 4; ++it) {
    float f = 0.f, fp = 0.f;
#pragma unroll
    for (int k = 0; k < kTopGroups; ++k) {
      const float x = fmaxf(v[k] - t, 0.f);
      const float g = x > 0.f ? pow_rm1<AM>(x, r) : 0.f;
      f = fmaf(g, x, f);
      fp += g;
    }
    f += __shfl_xor(f, 32);
    fp += __shfl_xor(fp, 32);
    const bool up = f > 1.0f;  // (then fp > 0)
    if (__ballot(up) == 0ull) break;
    if (up) t += (f - 1.0f) / (r * fp);
  }
  // (entries of no key are about -3e38: a row whose a is so small that they could count keeps the bound it has)
  return a > 1.0e-30f ? fmaxf(lo, t - 4e-6f * fmaxf(1.0f, fabsf(t))) : lo;
}

// Counters only: how many different 32-key blocks the wave's lanes' first ne entries name.
template <int G>
__device__ __forceinline__ unsigned distinct_blocks(const TopGroups<G>& top, const GroupNumbers<G>& gn, int ne, int lane) {
  unsigned n = 0;
  int mine[kTopGroups];
#pragma unroll
  for (int k = 0; k < kTopGroups; ++k) mine[k] = k < ne ? (int)((__float_as_uint(top.t[k]) & ~gn.keep) / GroupNumbers<G>::kPerBlock) : -1;
#pragma unroll 1
  for (int l = 0; l < 64; ++l) {
#pragma unroll
    for (int k = 0; k < kTopGroups; ++k) {
      const int jb = __builtin_amdgcn_readlane(mine[k], l);
      if (jb < 0) continue;
      ++n;  // counted once: every lane's further entries of the block are struck out
#pragma unroll
      for (int e = 0; e < kTopGroups; ++e) mine[e] = mine[e] == jb ? -1 : mine[e];
    }
  }
  return n;
}

// Lanes that remember too few groups, up to kScanLanes of a block: every key their row sees is looked at, a quarter of them by each wave,
// and what the waves find is put together in the keys' order.  (32 such rows at a time on the matrix cores, the keys shared out to the waves,
// takes longer for the few that there are: n 1024 44 -> 56 us.)
constexpr int kScanLanes = 8;
struct ScanLds {
  int lost_of_wave[kWaves];  // and, above 16 bits, how many entries of the wave's other lanes name a group to rescore
  int lane[kScanLanes];  // thread of the workgroup
  float cut[kScanLanes], w[kScanLanes];
  int negated[kScanLanes];
  int found[kScanLanes][kWaves];
};
static_assert(sizeof(ScanLds) == kScanBytes, "its place in LDS");
// notes: [kScanLanes][kWaves][kCandCap] of LDS; kt_first: key tiles before it are not looked at
template <typename C, typename T, int D, int G>
__device__ __forceinline__ int scan_lanes(const FwdSparseArgs& A, const C& q, int nlost, int first_group, ScanLds* sl, uint2* notes) {
  using O = OctetScores<C, T, D, G>;
  constexpr int N = O::W == 1 ? 2 : 1;
  const Geom& g = A.g;
  const O o(q, g, A.Q, A.K);
  const int oct = q.lane >> 3;
#pragma unroll 1
  for (int x = 0; x < nlost; ++x) {
    const int id = __builtin_amdgcn_readfirstlane(sl->lane[x]);
    typename O::Row row[N];
    row[0] = o.row_of(q.qb * kBlockRows + (id >> 6) * 32 + (id & 31), sl->cut[x], sl->negated[x] != 0, sl->w[x]);
    if (N > 1) row[N - 1] = row[0];
    const int end = ((row[0].lim + 31) >> 5) * O::P;
    const int share = ((end - first_group + kWaves * 8 - 1) / (kWaves * 8)) * 8;
    const int from = first_group + q.wave * share, to = min(end, from + share);
    int total = 0;
#pragma unroll 1
    for (int n0 = from; n0 < to; n0 += 8 * N) {
      int j0[N];
#pragma unroll
      for (int u = 0; u < N; ++u) j0[u] = O::first_key(n0 + 8 * u + oct, (id >> 5) & 1);
#pragma unroll
      for (int r0 = 0; r0 < G; r0 += 8) {
        float d[N];
        o.eight(row, j0, r0, d);
#pragma unroll
        for (int u = 0; u < N; ++u) {
          const int j = o.key(j0[u], r0);
          const bool pass = n0 + 8 * u + oct < to && j < row[u].lim && d[u] > row[u].cut;
          const unsigned long long all = __ballot(pass);
          if (all == 0ull) continue;
          const int at = total + (int)__builtin_amdgcn_mbcnt_hi((unsigned)(all >> 32), __builtin_amdgcn_mbcnt_lo((unsigned)all, 0u));
          if (pass && at < kCandCap) notes[(x * kWaves + q.wave) * kCandCap + at] = make_uint2((unsigned)j, __float_as_uint(d[u]));
          total += (int)__popcll(all);
        }
      }
    }
    if (q.lane == 0) sl->found[x][q.wave] = total;
  }
  __syncthreads();
  int cnt = -1;  // the lane's own count, if it is one of them
#pragma unroll 1
  for (int x = 0; x < nlost; ++x) {
    const int id = sl->lane[x];
    int before = 0, total = 0;
#pragma unroll
    for (int w = 0; w < kWaves; ++w) {
      const int n = sl->found[x][w];
      if (w < q.wave) before += n;
      total += n;
    }
    uint2* list = A.cand + list_entry<kCandCap>(q.bh, A.nqb, q.qb, id >> 6, id & 63);
    if (q.lane < sl->found[x][q.wave] && before + q.lane < kCandCap)
      list[(before + q.lane) * kListStride] = notes[(x * kWaves + q.wave) * kCandCap + min(q.lane, kCandCap - 1)];
    if (id == q.tid) cnt = total;
  }
  return cnt;
}

// Groups to rescore in a wave up to which the second sweep is not taken: kStart and kPerTile for every 128 keys of the block, for short
// blocks kShort and 48 for every 128 keys (a sweep of few tiles is over before sixteen groups at a time are).  Measured, bf16 (list kernel, before the short
// blocks' line; never / 160 + 6 / 48 + 24 / 24 + 12): B 4, H 12, n 4096, alpha 1.25 220 / 195 / 221 / 196 us; per-query scales, B 3, n 1999, bias
// 128 / 109 / 128 / 108; B 8, n 1024, alpha 1.5 41 / 41 / 41 / 54; n 4096 93 / 94 / 93 / 98.  Forward, 160 + 6 t with 48 + 48 t / without / with
// 24 + 24 t: B 8, H 12, n 64 24.4 / 26.2 / 24.6, n 200 31.2 / 33.1 / 31.6, n 500 43.0 / 43.8 / 46.5; H 12, n 1024 53.8 / 54.2 / 60.3.  fp32 (forward,
// 96 + 48 t / 48 + 24 t / 24 + 12 t / always swept): B 2, H 12, n 300 60 / 70 / 70 / 70; B 8, n 600 85 / 103 / 111 / 111; n 4096 320 / 315 / 321 / 599;
// D 128, H 16, B 2, n 200 64 / 75 / 77 / 77; alpha 1.25, B 2, n 2000 676 / 672 / 700 / 704 (160 + 6 t 690).
template <typename T>
struct SweepAgain {
  static constexpr int kStart = 160;
  static constexpr int kPerTile = sizeof(T) == 2 ? 6 : 24;
  static constexpr int kShort = sizeof(T) == 2 ? 48 : 96;
  static __device__ __forceinline__ int most_groups(int keys) { return min(kStart + (keys >> 7) * kPerTile, kShort + (keys >> 7) * 48); }
};

// What follows the sweep over the scores of a block: the rows' bounds, the scores of the keys that can matter, the lists.
// m1: the lane's largest score; n_vis: blocks the wave computed; places: of the sweep's memory that were kept throughout.  All threads of the workgroup; the tile buffers are free.
template <typename C, typename T, int D, int AM, int G, int LS, bool RING>
__device__ __forceinline__ void make_lists(const FwdSparseArgs& A, const C& q, TopGroups<G>& top, float m1, char* smem, int strip_no,
                                           unsigned n_vis, int places) {
  const Geom& g = A.g;
  int* ovf = reinterpret_cast<int*>(smem + ListCfg<T, D>::kFwdTiles);
  // (with the ring: in its third buffer, which sweeps of at most two tiles leave alone)
  char* lds_cells = ListCfg<T, D>::kRing ? smem + 2 * C::kTileBytes : smem + ListCfg<T, D>::kFwdTiles + kListHeaderBytes + sizeof(ScanLds);
  const GroupNumbers<G> gn(g.Nk);
  const int flag_idx = q.bh * A.nqb + q.qb;
  const long long row_idx = (long long)q.bh * g.Nq + (q.valid ? q.i : 0);
  const bool live = q.valid && q.lim > 0;
  const float r = 1.0f / (g.alpha - 1.0f);
  m1 = fmaxf(m1, __shfl_xor(m1, 32));
  const float m2 = top.runner_up(gn);
  const float y1 = live ? q.a * m1 : 0.f;
  float lo = y1 - 1.0f;  // App. A eq. (bounds), left end
  float hi = live ? y1 - __builtin_amdgcn_exp2f(-(g.alpha - 1.0f) * __builtin_amdgcn_logf((float)q.lim)) : 0.f;
  // two-element sub-problem {y1, y2}: its threshold is a lower bound of the row's
  if (live && m2 > -2.9e38f) lo = two_key_bound<AM>(y1, q.a * m2, r);
  // Rows of at most three blocks keep the two-key bound: in a dense head the tighter one keeps some first blocks, whose rows are that short, on
  // long lists, and the launch then waits for the finish kernel's long tail and for the tiled kernel, which the head's other blocks
  // need anyway.  Training steps with the limit / without: B 2, H 12, dense rows, n 256 93 / 142 us, n 300 108 / 154, n 500 135 / 182; B 8, n 128
  // 134 / 157.  Rows without a scale, which all fit the lists, pay for it: n 96 112 / 100, n 128 124 / 113, forward n 64 40 / 36.
  if (live && q.lim > 96) lo = top_groups_bound<AM>(top, gn, q.a, lo, r);
  lo = fminf(lo, hi);
  const float cut = raw_cut(q.a, live, lo);

  // A lane whose last place is above the cut may have lost groups that count.  Where there are few of them in the block all their
  // keys are looked at (scan_lanes()); where there are more, a second sweep over the scores of the block finds the keys of all its rows.  (With
  // the other lanes' groups rescored all the same, and only the lost ones looked for in the sweep, the longest workgroups had both in turn: forward, 12 heads,
  // alpha 1.25, B 2, n 1999 236 -> 221 us, with distance bias 257 -> 242, B 4, n 4096 402 -> 391.)
  int first = 0;
  if constexpr (C::BIAS) first = q.kt_first_wave * C::NSB;
  const int seen = (((q.wave_lim_max + 31) >> 5) - first) * GroupNumbers<G>::kPerBlock;
  int ne = live ? top.above(cut, gn) : 0;
  bool lost = ne >= places && seen > places;
  const unsigned long long lost_lanes = __ballot(lost);
  ScanLds* sl = reinterpret_cast<ScanLds*>(ovf + kListHeaderBytes / 4);
  int items = 0;  // at most 64 kTopGroups
#pragma unroll
  for (int k = 0; k < 4; ++k) items += (int)__popcll(__ballot(!lost && ((ne >> k) & 1) != 0)) << k;
  if (q.lane == 0) sl->lost_of_wave[q.wave] = (int)__popcll(lost_lanes) | items << 16;
  __syncthreads();  // (also: the tile buffers are free)
  int lost_before = 0, nlost = 0, most = 0;
#pragma unroll
  for (int w = 0; w < kWaves; ++w) {
    const int n = sl->lost_of_wave[w];
    if (w < q.wave) lost_before += n & 0xffff;
    nlost += n & 0xffff;
    most = max(most, n >> 16);
  }
  nlost = __builtin_amdgcn_readfirstlane(nlost);
  most = __builtin_amdgcn_readfirstlane(most);
  // Rescoring goes by the wave with the most groups, the second sweep by the keys: in short rows that keep many keys the sweep is cheaper.
  const bool again = nlost > kScanLanes || most > SweepAgain<T>::most_groups(q.block_lim - first * 32);
  if (lost && !again) {
    const int x = lost_before + (int)__builtin_amdgcn_mbcnt_hi((unsigned)(lost_lanes >> 32), __builtin_amdgcn_mbcnt_lo((unsigned)lost_lanes, 0u));
    sl->lane[x] = q.tid;
    sl->cut[x] = cut;
    sl->negated[x] = q.c < 0.f ? 1 : 0;
    if constexpr (C::BIAS) sl->w[x] = q.w; else sl->w[x] = 0.f;
  }
  if (lost) ne = 0;
  uint2* wave_list = A.cand + list_entry<kCandCap>(q.bh, A.nqb, q.qb, q.wave, 0);
  int cnt = 0;
  unsigned n_qk2 = 0, n_cand_tiles = 0;
  // The cutoff comes from the matrix cores' scores, and what is compared with it from sums in another order.  Where the products are some 1e5
  // times the bracket's width the two may differ by as much, and none of a row's keys pass: the block is the tiled kernel's, whose scores are
  // the sweep's.  (A list that is not empty holds the row's largest score.  Rows of infinite or NaN scores have no list.)
  auto none_passed = [&](bool looked_at) {
    const bool finite = m1 > -2.9e38f && fabsf(lo) < 3.0e38f;
    return __ballot(looked_at && live && finite && cnt + __shfl_xor(cnt, 32) == 0) != 0ull;
  };
  bool fits;
  if (again) {
    C qs = q;  // (its fragments and offsets are loaded again: kept through what comes before they would be spilled; scale and window
               // are kept: with them made again too the kernel of B 4, H 12, n 4096, alpha 1.25 took 190 us instead of 185)
    qs.load_fragments(g, A.Q);
    fits = collect_sweep<C, T, D, kCandCap, LS, RING>(qs, g, A.K, smem, ovf, lds_cells, cut, A.cells, wave_list + q.lane, cnt, n_qk2, n_cand_tiles,
                                                __ballot(live) != 0ull, strip_no);
  } else {
    if (A.stats) n_cand_tiles = distinct_blocks<G>(top, gn, lost ? places : ne, q.lane);
    if (!rescore_groups<C, T, D, G>(q, g, A.Q, A.K, top, gn, cut, ne, reinterpret_cast<int*>(smem) + q.wave * kRescoreWords, wave_list, cnt))
      ovf[2] = 1;
    if (none_passed((((lost_lanes | lost_lanes >> 32 | lost_lanes << 32) >> q.lane) & 1ull) == 0ull)) ovf[2] = 1;
    if (nlost > 0) {
      __syncthreads();
      if (ovf[2] == 0) {
        const int found = scan_lanes<C, T, D, G>(A, q, nlost, first * GroupNumbers<G>::kPerBlock, sl, reinterpret_cast<uint2*>(smem));
        if (found >= 0) {
          if (found > kCandCap) ovf[2] = 1;
          cnt = min(found, kCandCap);
          if (A.stats) atomicAdd(&A.stats[ENTMAX_STAT_FWD_CAND_TILES], (unsigned long long)max(cnt - places, 0));  // (at most)
        }
        if (none_passed(true)) ovf[2] = 1;
      }
    }
    pool_want(ovf + 3, cnt, q.lane);
    __syncthreads();
    fits = ovf[2] == 0;
  }
  if (!fits) {
    // the tiled kernel takes the block, and with it what the sweep found out about every row
    if (q.tid == 0) A.dense_flag[flag_idx] = kFlagWithBounds;
    if (q.valid && q.hh == 0) A.bounds[row_idx] = make_float2(lo, y1);
  } else {
    if (q.tid == 0) A.dense_flag[flag_idx] = -ovf[3];
    if (q.valid) {
      A.lcnt[row_idx * 2 + q.hh] = cnt;
      if (q.hh == 0) A.bounds[row_idx] = make_float2(lo, hi);
    }
  }
  if (A.stats && q.lane == 0) {
    const unsigned n_win = q.window_skipped_blocks();
    atomicAdd(&A.stats[ENTMAX_STAT_FWD_TILES_VISIBLE], (unsigned long long)(n_vis + n_win));
    if (C::BIAS) atomicAdd(&A.stats[ENTMAX_STAT_FWD_WINDOW_SKIPPED], (unsigned long long)n_win);
    atomicAdd(&A.stats[ENTMAX_STAT_FWD_LIST_QK], (unsigned long long)(n_vis + n_qk2));
    if (fits) {
      atomicAdd(&A.stats[ENTMAX_STAT_FWD_CAND_TILES], (unsigned long long)n_cand_tiles);
      if (q.wave == 0) atomicAdd(&A.stats[ENTMAX_STAT_FWD_SPARSE_BLOCKS], 1ull);
    }
  }
}

// The sweep over the scores and what follows it, for R adjacent query blocks from block blk on: every wave holds its 32-row
// group of each of them, so that with two a K fragment read from LDS feeds two matrix instructions and a K tile staged
// through LDS serves 256 rows.
// One sweep and rescored groups instead of two sweeps (kernel time, causal, alpha 1.5): B 8, H 12, n 1024, D 64 47 -> 41 us; B 4, H 12,
// n 4096 136 -> 94; B 2, H 16, n 8192, D 128 530 -> 357; B 1, H 12, n 32768 (two blocks a workgroup) 1275 -> 880; B 2, H 16, n 5003,
// D 128, alpha 2 245 -> 150.  Of the 94 us the sweep is 57 (its matrix instructions alone would take 21, its vector instructions 25: a
// SIMD's three waves share one issue slot, and alone on its CU a workgroup needs 0.7 us a tile), the rescoring 21.  What was in the way before: the second sweep's branches around every block with a candidate (82 us).
// Sixteen keys a group instead of eight: the sweep 6 us less, the rescoring's reads doubled, 94 -> 104 us.
template <typename T, int D, int AM, bool BIAS, int R>
__device__ __forceinline__ void fwd_lists_blocks(const FwdSparseArgs& A, int bh_, int blk, char* smem, int strip_no) {
  using C = QCtx<T, D, ListCfg<T, D>::kTile, BIAS>;
  using Cfg = ListCfg<T, D>;
  using KTile = typename C::KTile;
  constexpr int KT = C::KT, NSB = C::NSB, NC = C::NC;
  const Geom& g = A.g;
  int* ovf = reinterpret_cast<int*>(smem + Cfg::kFwdTiles);  // sticky overflow flags: [0], [1] by tile parity, [2] list; [3] pool_want()
  int* votes = ovf + 4;                                      // the waves' votes (see below)
  const int tid = threadIdx.x;
  if (tid < kListHeaderBytes / 4) ovf[tid] = 0;  // (first barrier: init_window's or the sweep's)

  C q[R];
#pragma unroll
  for (int k = 0; k < R; ++k) {
    q[k].init(g, A.Q, bh_, blk + k);
    q[k].init_window(g);
  }
  if (q[R - 1].block_lim == 0) {  // no row of any block sees any key: the finish kernel writes the zeros
#pragma unroll
    for (int k = 0; k < R; ++k) {
      const long long row_idx = (long long)q[k].bh * g.Nq + (q[k].valid ? q[k].i : 0);
      if (q[k].valid) {
        A.lcnt[row_idx * 2 + q[k].hh] = 0;
        if (q[k].hh == 0) A.bounds[row_idx] = make_float2(0.f, 0.f);
      }
      if (tid == 0) A.dense_flag[q[k].bh * A.nqb + q[k].qb] = 0;
    }
    return;
  }
  // tiles first .. ntiles - 1, those before whole_end wholly visible to every row
  const int ntiles = q[R - 1].ntiles;  // a later block sees at least the keys of the earlier one
  const int whole_end = __builtin_amdgcn_readfirstlane(row_limit(g, q[0].qb * kBlockRows) / KT);
  int first = 0;
  bool biased = false;  // (of the head: the same for all waves)
  if constexpr (BIAS) {
    first = q[0].kt_first;
#pragma unroll
    for (int k = 1; k < R; ++k) first = min(first, q[k].kt_first);
#pragma unroll
    for (int k = 0; k < R; ++k) q[k].kt_first = q[k].kt_first_wave = first;  // (the waves go through the tiles together)
    biased = g.slopes[q[0].h] != 0.f;
  }
  Slot slots[1];
  slots[0].base = reinterpret_cast<const char*>(reinterpret_cast<const T*>(A.K) + (long long)q[0].b * g.kv_sb +
                                                (long long)q[0].h * g.kv_sh);
  slots[0].row_bytes = g.kv_sn * (long long)sizeof(T);

  const GroupNumbers<Cfg::kGroup> gn(g.Nk);
  using Top = TopGroups<Cfg::kGroup>;
  Top top[R];
  float m1[R];
#pragma unroll
  for (int k = 0; k < R; ++k) {
    top[k].init();
    m1[k] = -kInf;
  }

  // Dense rows are found out on the first tile: where, for three quarters of a wave's rows, half of the keys of
  // the tile's first block come within the bracket's width of the block's largest score, the lists would overflow anyway (a row of
  // the paper's sparse setting has a handful of such keys).  Blocks all of whose waves vote so are handed to the
  // tiled kernel after that one block of scores (fp32: two tiles) instead of after a full sweep (a matter of time only: the tiled
  // kernel handles any row).  In a head's ragged last block the rows that there are decide, and as its lists have less to hold, three quarters of the keys
  // are asked for: training steps, B 2, H 12, dense rows, n 300 170 -> 109 us (fp32 328 -> 255), n 500 163 -> 134; 8 heads, n 627, alpha 1.25,
  // no scale 154 -> 141; with half of the keys there too B 8, H 12, n 160, no scale 135 -> 162.
  auto vote = [&](const C& qk, const f32x16_t& acc, float lm) -> bool {
    // the bracket's width in raw units, a little wider than needed (rounding)
    const float reach = (qk.valid && qk.lim > 0) ? (qk.a > 0.f ? 1.0001f / qk.a : 3.0e38f) : -kInf;
    int near = 0;  // of the lane's 16 keys of the tile's first block
    const int enough = (qk.qb + 1) * kBlockRows > g.Nq ? 12 : 8;
#pragma unroll
    for (int e = 0; e < 16; ++e) near += (acc[e] + reach > lm) ? 1 : 0;
    return 4 * (int)__popcll(__ballot(near >= enough)) >= 3 * (int)__popcll(__ballot(qk.valid && qk.lim > 0));
  };
  auto all_dense = [&]() { return (votes[0] & votes[1] & votes[2] & votes[3]) != 0; };
  auto vote_on = [&](int kt, const char* tl) {
    bool dense = true;
#pragma unroll
    for (int k = 0; k < R; ++k) {
      const f32x16_t acc = q[k].scores(tl, 0, kt);
      dense = vote(q[k], acc, max16(acc)) && dense;
    }
    if (dense && q[0].lane == 0) votes[q[0].wave] = 1;
  };
  // any tile, one 32-key block after the other
  auto general = [&](int kt, const char* tl) {
    if (!Cfg::kRing && kt == first && kt < whole_end) vote_on(kt, tl);
#pragma unroll 1
    for (int sb = 0; sb < NSB; ++sb) {
      const int j0 = kt * KT + sb * 32;
#pragma unroll
      for (int k = 0; k < R; ++k) {
        if (j0 >= q[k].wave_lim_max) continue;
        f32x16_t acc = q[k].scores(tl, sb, kt);
        if (j0 + 32 > q[k].wave_lim_min) mask_block(q[k], acc, j0);
        m1[k] = fmaxf(m1[k], top[k].take(acc, gn, kt * NSB + sb));
      }
    }
  };
  int places = kTopGroups;
  if constexpr (!Cfg::kRing) {
    sweep_tiles<C, T, D, 1, 0, Cfg::kDepth>(
        smem, slots, ntiles, g.Nk, tid, [&](int kt) { return kt >= first; }, general,
        // (the votes of a tile are final before the barrier that ends it)
        [&](int kt) { return kt == first + 1 && all_dense(); });
  } else {
    TileRing<C, T, D> ring;
    ring.start(smem, slots[0], first, ntiles, g.Nk);
    // Tiles all of whose keys every row sees.  The matrix instructions of a block run beside the vector work on the scores of
    // the one before it (with two query blocks: of the other query block), which needs two accumulators; the last one waits
    // over the barrier for the next tile.  A K fragment is requested when the one before it in its place has been used.
    auto whole_tiles = [&](auto biased_, auto places_) {
      constexpr int K = decltype(places_)::value;
      f32x16_t late;
#pragma unroll
      for (int e = 0; e < 16; ++e) late[e] = -kInf;
      int late_jb = 0;
      float late_floor = Top::kNothing;  // (nothing waits)
      auto pipelined = [&](int kt, const char* tl) {
        constexpr int F = 4;  // fragments in registers
        Frag<T> kf[F];
#pragma unroll
        for (int cc = 0; cc < F; ++cc) kf[cc] = q[0].koff[cc].load(tl, 0);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int sb = 0; sb < NSB; ++sb) {
#pragma unroll
          for (int k = 0; k < R; ++k) {
            const int kl = k == 0 ? R - 1 : k - 1;  // the query block whose scores wait
            const int j0 = kt * KT + sb * 32;
            float m[Top::Numbers::kPerBlock], x[Top::Numbers::kPerBlock];
            f32x16_t acc = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
            if constexpr (decltype(biased_)::value) q[k].bias_before(acc, j0);
#pragma unroll
            for (int cc = 0; cc < NC; ++cc) {
              acc = Elem<T>::mma(kf[cc % F], q[k].qf[cc], acc);
              // what this place holds next: a later fragment of the block, its first ones again, or the next block's
              const int nx = cc + F;
              if (nx < NC)
                kf[cc % F] = q[0].koff[nx].load(tl, sb * 32 * KTile::kRowBytes);
              else if (k + 1 < R) {
                if (NC > F) kf[cc % F] = q[0].koff[nx - NC].load(tl, sb * 32 * KTile::kRowBytes);
              } else if (sb + 1 < NSB)
                kf[cc % F] = q[0].koff[nx - NC].load(tl, (sb + 1) * 32 * KTile::kRowBytes);
              __builtin_amdgcn_sched_barrier(0);  // (the order is the point: left to itself the compiler issues all products first)
              if (cc == 0) top[kl].template take_part<0, K>(late, gn, late_jb, late_floor, m, x, m1[kl]);
              if (cc == NC / 4) top[kl].template take_part<1, K>(late, gn, late_jb, late_floor, m, x, m1[kl]);
              if (cc == 2 * NC / 4) top[kl].template take_part<2, K>(late, gn, late_jb, late_floor, m, x, m1[kl]);
              if (cc == 3 * NC / 4) top[kl].template take_part<3, K>(late, gn, late_jb, late_floor, m, x, m1[kl]);
              __builtin_amdgcn_sched_barrier(0);
            }
            late = acc;
            late_jb = j0 >> 5;
            late_floor = Top::kFloor;
          }
        }
#pragma unroll
        for (int k = 0; k < R; ++k) {  // (all of it happens here: the compiler moves what it can behind the next branch)
#pragma unroll
          for (int e = 0; e < K; ++e) asm volatile("" : "+v"(top[k].t[e]));
          asm volatile("" : "+v"(m1[k]));
        }
      };
#pragma unroll 1
      while (ring.kt < whole_end) {
        ring.step([&](const char* tl) { pipelined(ring.kt, tl); });
      }
      m1[R - 1] = fmaxf(m1[R - 1], top[R - 1].take(late, gn, late_jb, late_floor));
    };
    bool weak = false;
#pragma unroll
    for (int k = 0; k < R; ++k)
      weak = weak || (q[k].valid && q[k].lim > 0 && !(q[k].a * sqrtf((float)D) >= kFewPlacesScale));
    if (__ballot(weak) == 0ull) places = kFewPlaces;
    auto both = [&](auto biased_) {
      if (places == kFewPlaces)
        whole_tiles(biased_, std::integral_constant<int, kFewPlaces>());
      else
        whole_tiles(biased_, std::integral_constant<int, kTopGroups>());
    };
    if (first < whole_end) {
      vote_on(first, smem);
      __syncthreads();
    }
    if (all_dense()) {
      ring.abandon();
    } else {
      if (!BIAS || !biased) {
        both(std::false_type());
      } else if constexpr (BIAS) {
        if (g.causal) both(std::true_type());  // (every key of such a tile lies at or before every row's position)
      }
      while (ring.kt < ntiles) ring.step([&](const char* tl) { general(ring.kt, tl); });
    }
  }
  // blocks the waves have computed
  unsigned n_vis[R];
#pragma unroll
  for (int k = 0; k < R; ++k) n_vis[k] = (unsigned)max(((q[k].wave_lim_max + 31) >> 5) - first * NSB, 0);
  if (all_dense()) {  // (the sweep ended on a barrier)
    __syncthreads();  // every thread has read the votes before the next block's zeroes them
#pragma unroll
    for (int k = 0; k < R; ++k) {
      if (tid == 0) A.dense_flag[q[k].bh * A.nqb + q[k].qb] = kFlagDense;
      if (A.stats && q[k].lane == 0)
        atomicAdd(&A.stats[ENTMAX_STAT_FWD_LIST_QK], (unsigned long long)Cfg::kRing ? 1ull : (unsigned long long)min(n_vis[k], 2u * NSB));
    }
    return;
  }
  if constexpr (R == 1) {
    make_lists<C, T, D, AM, Cfg::kGroup, Cfg::kRing ? Cfg::kThirdBufferCells : Cfg::kFwdCells, Cfg::kRing>(A, q[0], top[0], m1[0], smem, strip_no, n_vis[0], places);
  } else {
    // What is left is done for one block after the other; what the sweep found out about the second waits in LDS, in the third
    // tile buffer (which nothing else uses now), so that only one block's rows are in registers.
    static_assert(Cfg::kRing && R == 2 && kTopGroups * kThreads * 4 <= C::kTileBytes, "a tile buffer holds a block's entries");
    float* stash = reinterpret_cast<float*>(smem + 2 * C::kTileBytes) + tid;  // [kTopGroups][kThreads]
    Top tk = top[0];
#pragma unroll
    for (int e = 0; e < kTopGroups; ++e) stash[e * kThreads] = top[1].t[e];
    const float m_first = m1[0], m_last = m1[R - 1];
    const unsigned n_first = n_vis[0], n_last = n_vis[R - 1];
#pragma unroll 1
    for (int k = 0; k < R; ++k) {
      if (k) {
        __syncthreads();  // (every thread is done with the first block's words)
        if (tid < kListHeaderBytes / 4) ovf[tid] = 0;
        __syncthreads();
      }
      C qk;
      qk.init(g, A.Q, bh_, blk + k);
      if constexpr (BIAS) qk.kt_first = qk.kt_first_wave = first;
      if (k) {
#pragma unroll
        for (int e = 0; e < kTopGroups; ++e) tk.t[e] = stash[e * kThreads];
      }
      make_lists<C, T, D, AM, Cfg::kGroup, Cfg::kFwdCells, false>(A, qk, tk, k ? m_last : m_first, smem, strip_no + k, k ? n_last : n_first, places);
    }
  }
}

template <typename T, int D, int AM, bool BIAS>
__global__ __launch_bounds__(kThreads, (ListCfg<T, D>::kFwdOcc)) void fwd_lists_kernel(FwdSparseArgs A) {
  extern __shared__ __attribute__((aligned(16))) char smem[];
  PairItem it;
  if (A.unpaired) {  // a head's blocks on one XCD, the longest first
    const int item = xcd_remap(blockIdx.x, gridDim.x);
    it.bh = __builtin_amdgcn_readfirstlane(item / A.nqb);
    it.first = A.nqb - 1 - __builtin_amdgcn_readfirstlane(item % A.nqb);
    it.second = -1;
  } else {
    it = pair_item(A.nqb);
  }
  if (blockIdx.x == 0 && threadIdx.x == 0) {
    A.dense_flag[A.g.B * A.g.H * A.nqb] = 0;
  }
  if (blockIdx.x == 0 && A.pool_cursor && (int)threadIdx.x < (1 << A.pool_shift))
    *reinterpret_cast<unsigned long long*>(A.pool_cursor + (size_t)threadIdx.x * kSavedCursorStride) = 0ull;
  if (A.kcount) {
    // this workgroup's share of its head's per-key counters starts at zero for the finish kernel
    const int npair = A.unpaired ? A.nqb : (A.nqb + 1) >> 1, pp = A.nqb - 1 - it.first;
    const int chunk = (A.g.Nk + npair - 1) / npair;
    int* dst = A.kcount + (long long)it.bh * A.g.Nk;
    for (int j = pp * chunk + (int)threadIdx.x; j < min(A.g.Nk, (pp + 1) * chunk); j += kThreads) dst[j] = 0;
  }
  for (int part = 0; part < 2; ++part) {
    const int blk = part ? it.second : it.first;
    if (blk < 0) break;
    if (part) __syncthreads();
    fwd_lists_blocks<T, D, AM, BIAS, 1>(A, it.bh, blk, smem, (int)blockIdx.x);
  }
}

// ------------------------------------------------- long sequences: two query blocks per workgroup
// Used where the launch still fills the chip with half as many workgroups (Nk >= ListCfg::kPairMinKeys).
template <typename T, int D, int AM, bool BIAS>
__global__ __launch_bounds__(kThreads, (ListCfg<T, D>::kFwdOcc)) void fwd_lists_pair_kernel(FwdSparseArgs A) {
  extern __shared__ __attribute__((aligned(16))) char smem[];
  const int nsb = (A.nqb + 1) >> 1;  // pairs of adjacent blocks per head
  const PairItem it = pair_item(nsb);
  if (blockIdx.x == 0 && threadIdx.x == 0) A.dense_flag[A.g.B * A.g.H * A.nqb] = 0;
  if (blockIdx.x == 0 && A.pool_cursor && (int)threadIdx.x < (1 << A.pool_shift))
    *reinterpret_cast<unsigned long long*>(A.pool_cursor + (size_t)threadIdx.x * kSavedCursorStride) = 0ull;
  if (A.kcount) {
    // this workgroup's share of its head's per-key counters starts at zero for the finish kernel
    const int npair = (nsb + 1) >> 1, pp = nsb - 1 - it.first;
    const int chunk = (A.g.Nk + npair - 1) / npair;
    int* dst = A.kcount + (long long)it.bh * A.g.Nk;
    for (int j = pp * chunk + (int)threadIdx.x; j < min(A.g.Nk, (pp + 1) * chunk); j += kThreads) dst[j] = 0;
  }
  for (int part = 0; part < 2; ++part) {
    const int sblk = part ? it.second : it.first;
    if (sblk < 0) break;
    if (part) __syncthreads();
    if (2 * sblk + 1 < A.nqb)
      fwd_lists_blocks<T, D, AM, BIAS, 2>(A, it.bh, 2 * sblk, smem, 2 * (int)blockIdx.x);
    else  // a head's odd last block
      fwd_lists_blocks<T, D, AM, BIAS, 1>(A, it.bh, 2 * sblk, smem, 2 * (int)blockIdx.x);
  }
}

// widen 8 (bf16) or 4 (fp32) consecutive elements to fp32
template <typename T>
__device__ __forceinline__ void load_row_f32(const T* row, int n, float* out) {
  if constexpr (sizeof(T) == 2) {
#pragma unroll
    for (int c8 = 0; c8 < n / 8; ++c8) {
      u32x4_t w = *reinterpret_cast<const u32x4_t*>(row + 8 * c8);
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        out[8 * c8 + 2 * k] = __uint_as_float(w[k] << 16);
        out[8 * c8 + 2 * k + 1] = __uint_as_float(w[k] & 0xffff0000u);
      }
    }
  } else {
#pragma unroll
    for (int c4 = 0; c4 < n / 4; ++c4) {
      f32x4_t w = *reinterpret_cast<const f32x4_t*>(row + 4 * c4);
#pragma unroll
      for (int k = 0; k < 4; ++k) out[4 * c4 + k] = w[k];
    }
  }
}
// The same row kept as loaded (16-byte words) and widened only where it is used: a gather in flight
// costs half (bf16) of the registers of a widened row.
template <typename T, int N>
struct RawRow {
  static constexpr int kWords = N * (int)sizeof(T) / 16;
  u32x4_t w[kWords];
  __device__ __forceinline__ void load(const T* row) {
#pragma unroll
    for (int c = 0; c < kWords; ++c) w[c] = *reinterpret_cast<const u32x4_t*>(reinterpret_cast<const char*>(row) + 16 * c);
  }
  // element t (a compile-time index once the caller's loop is unrolled)
  __device__ __forceinline__ float get(int t) const {
    if constexpr (sizeof(T) == 2) {
      const uint32_t word = w[t >> 3][(t >> 1) & 3];
      return __uint_as_float((t & 1) ? (word & 0xffff0000u) : (word << 16));
    } else {
      return __uint_as_float(w[t >> 2][t & 3]);
    }
  }
};

// element t of a 16-byte word of a row, widened
template <typename T>
__device__ __forceinline__ float word_elem(const u32x4_t& w, int t) {
  if constexpr (sizeof(T) == 2)
    return __uint_as_float((t & 1) ? (w[t >> 1] & 0xffff0000u) : (w[t >> 1] << 16));
  else
    return __uint_as_float(w[t]);
}

template <typename T>
__device__ __forceinline__ void store_row(T* row, int n, const float* v) {
  if constexpr (sizeof(T) == 2) {
#pragma unroll
    for (int c8 = 0; c8 < n / 8; ++c8) *reinterpret_cast<u32x4_t*>(row + 8 * c8) = Elem<T>::pack(v + 8 * c8).v;
  } else {
#pragma unroll
    for (int c4 = 0; c4 < n / 4; ++c4)
      *reinterpret_cast<f32x4_t*>(row + 4 * c4) = f32x4_t{v[4 * c4], v[4 * c4 + 1], v[4 * c4 + 2], v[4 * c4 + 3]};
  }
}

// Row coordinates of a lane in the list kernels: wave w of block qb owns rows qb*128 + 32 w .. + 31, lane l row (l % 32), list half
// hh = l / 32 -- the same assignment as in the sweeps that wrote the lists; a workgroup is one 128-row block.  With `groups`
// it is one of the block's four 32-row groups, which all four waves then have.
// (li, w32): the row's lane and 32-row group in the sweeps' numbering, as list_entry() wants them.
// Where the heads divide evenly over the eight XCDs the workgroups are renumbered so that a head's rows all run on
// one XCD, the one whose L2 saw the head's keys and lists in the sweeps (finish kernel, measured on one box:
// B 4, H 12, n 4096: 54 -> 50 us; with 12 heads at n 32768, one and a half heads per XCD, it was 60 -> 73 us).
struct RowLane {
  int bh, b, h, qb, i, li, hh, w32;
  bool valid;
  __device__ __forceinline__ void init(const Geom& g, int nqb, bool groups = false) {
    const int tid = threadIdx.x, lane = tid & 63, per_block = groups ? kWaves : 1;
    const int vb = (g.B * g.H) % 8 == 0 ? xcd_remap(blockIdx.x, g.B * g.H * nqb * per_block) : (int)blockIdx.x;
    const int blk = vb / per_block;
    bh = blk / nqb;
    qb = blk % nqb;
    b = bh / g.H;
    h = bh % g.H;
    hh = lane >> 5;
    li = lane & 31;
    w32 = groups ? vb % per_block : tid >> 6;
    i = qb * kBlockRows + w32 * 32 + li;
    valid = i < g.Nq;
  }
};

template <typename T, int D, int AM>
__global__ __launch_bounds__(kThreads) void fwd_finish_kernel(FwdSparseArgs A) {
  const Geom& g = A.g;
  if ((int)blockIdx.x >= g.B * g.H * A.nqb) {  // riders behind the row workgroups
    transpose_ride<T, D>(A.ride, (int)blockIdx.x - g.B * g.H * A.nqb);
    return;
  }
  RowLane rl;
  rl.init(g, A.nqb);
  // (the flag is tested further down: every load that does not depend on another is issued first)
  const int blk = rl.bh * A.nqb + rl.qb;
  const int block_word = A.dense_flag[blk];
  // the blocks that share this one's part of the pool: block b of run r (a run: as many blocks as parts) is in part
  // (b + r) modulo the parts, so that a part's blocks are at all places of their heads; lane l looks at run l first
  const int my_run = blk >> A.pool_shift, pool_mask = (1 << A.pool_shift) - 1, part = (blk + my_run) & pool_mask;
  auto part_word = [&](int run) -> int {
    const long long other = ((long long)run << A.pool_shift) + ((part - run) & pool_mask);
    return other < (long long)g.B * g.H * A.nqb ? A.dense_flag[other] : 0;
  };
  const int first_part_word = A.list ? part_word(threadIdx.x & 63) : 0;
  constexpr int DH = D / 2;
  const float r = 1.0f / (g.alpha - 1.0f);
  const long long row_idx = (long long)rl.bh * g.Nq + (rl.valid ? rl.i : 0);
  const int lim = rl.valid ? row_limit(g, rl.i) : 0;
  const bool live = rl.valid && lim > 0;
  const float scale = rl.valid ? row_scale(g, rl.b, rl.h, rl.i, lim, nullptr, nullptr, nullptr) : 0.f;
  const float c = scale * (1.0f / sqrtf((float)D));
  const float a = (g.alpha - 1.0f) * fabsf(c);  // same arithmetic as the sweeps that made the lists
  const int cnt_raw = A.lcnt[row_idx * 2 + rl.hh];
  const float2 bd_raw = A.bounds[row_idx];
  const int cnt = live ? cnt_raw : 0;
  const float2 bd = live ? bd_raw : make_float2(0.f, 0.f);
  const uint2* mylist = A.cand + list_entry<kCandCap>(rl.bh, A.nqb, rl.qb, threadIdx.x >> 6, threadIdx.x & 63);
  const T* Vbh = reinterpret_cast<const T*>(A.V) + (long long)rl.b * g.kv_sb + (long long)rl.h * g.kv_sh;
  float lo = bd.x, hi = bd.y, tau = bd.x;
  unsigned n_support = 0;
  // the first entries are requested before the list length is known (the slots exist whatever they hold):
  // one memory round trip less on the critical path of this latency-bound kernel
  constexpr int kEarly = 4;
  uint2 early[kEarly];
#pragma unroll
  for (int e = 0; e < kEarly; ++e) early[e] = mylist[e * kListStride];
  if (block_word > 0) {  // the tiled kernel owns this block, and so do the backward's tiled kernels
    if (A.list && threadIdx.x == 0) A.bwd_flag[blk] = kBlockNoLists;
    if (threadIdx.x == 0) {
      int* count = A.dense_flag + g.B * g.H * A.nqb;
      const int slot = atomicAdd(count, 1);
      if (slot < kSplitMaxBlocks) count[1 + slot] = blk;
    }
    return;
  }
  // The 32-row group's piece of the pool, sized before the supports are known (see pool_want()).  Whether a block gets
  // one is settled by the blocks' wants alone: the blocks that share its part of the pool are counted in turn, first those whose
  // lists are sure to be used, then those whose supports may turn out too long for the backward, and it does while
  // the part holds what has been counted.  So the outputs do not depend on the order in which the workgroups run, and
  // blocks that the backward cannot use take no room from blocks that are sure to be used.  (By arrival, B 3, H 12, n 3081
  // with per-query scales kept 115 to 117 blocks on the backward's lists, dQ differing by 1.3e-3 between calls; so it
  // keeps the same 159.  The kernel itself: 44.1 -> 44.4 us at B 4, H 12, n 4096, D 64.)  Where in the part a group's piece lies is
  // without effect and left to a returning atomic.
  uint2* suplist = nullptr;
  int sup_off = 0;
  bool pool_full = false;
  if (A.list) {
    const int lane = threadIdx.x & 63;
    const bool my_long = (-block_word >> 16) != 0;
    auto counted_before = [&](int w, int run) -> int {  // entries of a block that is counted before this one
      const bool is_long = (-w >> 16) != 0;
      return w < 0 && (my_long ? !is_long || run < my_run : !is_long && run < my_run) ? -w & 0xffff : 0;
    };
    int ahead = counted_before(first_part_word, lane);
    for (int r0 = 64; r0 <= (g.B * g.H * A.nqb - 1) >> A.pool_shift; r0 += 64)  // (parts of more than 64 blocks)
      ahead += counted_before(part_word(r0 + lane), r0 + lane);
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) ahead += __shfl_xor(ahead, off);
    pool_full = (long long)ahead + (-block_word & 0xffff) > A.pool_part_cap;
    const int want = min(cnt, kBwdCap);
    int incl = want;  // inclusive running sum over the lanes
#pragma unroll
    for (int sft = 1; sft < 64; sft <<= 1) {
      const int up = __shfl_up(incl, sft);
      if (lane >= sft) incl += up;
    }
    const int total = __builtin_amdgcn_readlane(incl, 63);
    unsigned long long base = 0ull;
    if (lane == 0 && total > 0 && !pool_full)
      base = atomicAdd(reinterpret_cast<unsigned long long*>(A.pool_cursor + (size_t)part * kSavedCursorStride),
                       (unsigned long long)total);
    base = ((unsigned long long)(unsigned)__builtin_amdgcn_readfirstlane((int)(base >> 32)) << 32) |
           (unsigned)__builtin_amdgcn_readfirstlane((int)base);
    sup_off = pool_full ? 0 : (int)(part * A.pool_part_cap + (long long)base) + incl - want;
    if (!pool_full) suplist = A.list + sup_off;
  }
  int scnt = 0;  // support entries of this half row

  // NE: list entries per lane held in registers; chosen per wave from the longest list it holds.
  // (Same sums in the same order whichever NE is chosen: entry order.)
  auto finish = [&](auto ne_tag) {
    constexpr int NE = decltype(ne_tag)::value;
    float yv[NE], dvv[NE];
    unsigned jv[NE];
#pragma unroll
    for (int e = 0; e < NE; ++e) {
      uint2 en = make_uint2(0u, 0u);
      if (e < kEarly)
        en = early[e];
      else if (e < cnt)
        en = mylist[e * kListStride];
      jv[e] = (e < cnt) ? en.x : 0u;
      dvv[e] = __uint_as_float(en.y);
      yv[e] = (e < cnt) ? a * dvv[e] : -kInf;  // -inf: never positive
    }
    // entries beyond the NE held in registers (few lanes) are read again wherever they are needed
    const bool has_tail = __ballot(cnt > NE) != 0ull;
    bool done = !live;
    int iter = 0;
    float y_most = -kInf;
#pragma unroll
    for (int e = 0; e < NE; ++e) y_most = fmaxf(y_most, yv[e]);
    while (__ballot(!done) != 0ull && iter < kMaxSolveIters) {
      RowSums sums;
      sums.clear();
#pragma unroll
      for (int e = 0; e < NE; ++e) accumulate<AM>(sums, yv[e] - tau, r);
      if (has_tail)
        for (int e = NE; e < cnt; ++e) {
          const float y = a * __uint_as_float(mylist[e * kListStride].y);
          y_most = fmaxf(y_most, y);
          accumulate<AM>(sums, y - tau, r);
        }
      sums.combine_halves();
      if (iter == 0) {
        // The bracket is that of the list's scores.  Those of the sweep, which the bounds came from, are the same sums in another
        // order: with them a row of one key had p = 1 - 2 (a d_sweep - a d_list) (alpha 1.5) where it is 1.
        y_most = fmaxf(y_most, __shfl_xor(y_most, 32));
        if (y_most > -kInf) {
          lo = y_most - 1.0f;
          hi = y_most - __builtin_amdgcn_exp2f(-(g.alpha - 1.0f) * __builtin_amdgcn_logf((float)lim));
        }
      }
      if (!done) done = solve_step<AM>(sums, r, tau, lo, hi);
      ++iter;
    }
    // O = sum p_j v_j: each lane of a pair takes half of the features of every entry of the row
    float oacc[DH];
#pragma unroll
    for (int t = 0; t < DH; ++t) oacc[t] = 0.f;
#pragma unroll
    for (int e = 0; e < NE; ++e) {
      // (the same expression as the backward's row kernel, so that both sides agree on the support)
      float p_own = (live && e < cnt) ? pow_r<AM>(fmaxf(fmaf(dvv[e], a, -tau), 0.f), r) : 0.f;
      float p_oth = __shfl_xor(p_own, 32);
      unsigned j_oth = (unsigned)__shfl_xor((int)jv[e], 32);
      if (p_own > 0.f) {
        ++n_support;
        if (suplist && scnt < kBwdCap) {
          // (writing the entries after the gathers, so that the counter's answer is not waited for here, gained nothing)
          const unsigned rank = (unsigned)atomicAdd(&A.kcount[(long long)rl.bh * g.Nk + jv[e]], 1);
          suplist[scnt] = make_uint2(jv[e] | (min(rank, kSavedRankMost) << kSavedKeyBits), __float_as_uint(dvv[e]));
        }
        ++scnt;
      }
#pragma unroll
      for (int src = 0; src < 2; ++src) {
        // both lanes of the pair take the same entry: entry e of the lane whose half index is src
        float p = (rl.hh == src) ? p_own : p_oth;
        unsigned j = (rl.hh == src) ? jv[e] : j_oth;
        if (__ballot(p > 0.f) == 0ull) continue;
        if (p > 0.f) {
          RawRow<T, DH> vv;
          vv.load(Vbh + (long long)j * g.kv_sn + rl.hh * DH);
#pragma unroll
          for (int t = 0; t < DH; ++t) oacc[t] = fmaf(p, vv.get(t), oacc[t]);
        }
      }
    }
    if (has_tail) {
      for (int e = NE; __ballot(e < cnt) != 0ull; ++e) {
        uint2 en = make_uint2(0u, 0u);
        if (e < cnt) en = mylist[e * kListStride];
        float p_own = (live && e < cnt) ? pow_r<AM>(fmaxf(fmaf(__uint_as_float(en.y), a, -tau), 0.f), r) : 0.f;
        float p_oth = __shfl_xor(p_own, 32);
        unsigned j_oth = (unsigned)__shfl_xor((int)en.x, 32);
        if (p_own > 0.f) {
          ++n_support;
          if (suplist && scnt < kBwdCap) {
            const unsigned rank = (unsigned)atomicAdd(&A.kcount[(long long)rl.bh * g.Nk + en.x], 1);
            suplist[scnt] = make_uint2(en.x | (min(rank, kSavedRankMost) << kSavedKeyBits), en.y);
          }
          ++scnt;
        }
#pragma unroll
        for (int src = 0; src < 2; ++src) {
          float p = (rl.hh == src) ? p_own : p_oth;
          unsigned j = (rl.hh == src) ? en.x : j_oth;
          if (p > 0.f) {
            RawRow<T, DH> vv;
            vv.load(Vbh + (long long)j * g.kv_sn + rl.hh * DH);
#pragma unroll
            for (int t = 0; t < DH; ++t) oacc[t] = fmaf(p, vv.get(t), oacc[t]);
          }
        }
      }
    }
    if (rl.valid) {
      T* orow = reinterpret_cast<T*>(A.O) + (long long)rl.b * g.q_sb + (long long)rl.h * g.q_sh +
                (long long)rl.i * g.q_sn + rl.hh * DH;
      store_row<T>(orow, DH, oacc);
      if (rl.hh == 0) A.tau[row_idx] = live ? tau : 0.f;
      if (A.list) A.slcnt[row_idx * 2 + rl.hh] = (int)(((unsigned)sup_off << 5) | (unsigned)(pool_full ? 0 : min(scnt, kBwdCap)));
    }
  };
  if (__ballot(cnt > 4) == 0ull)
    finish(std::integral_constant<int, 4>());
  else
    finish(std::integral_constant<int, 8>());

  if (A.list) {
    // a support longer than the backward's lists hold, or no room left in the pool, sends the block to the
    // backward's tiled kernels
    const int any_long = __syncthreads_or(scnt > kBwdCap ? 1 : 0);
    if (threadIdx.x == 0) A.bwd_flag[blk] = pool_full ? kBlockNoLists : (any_long ? kBlockListsUnused : 0);
  }
  if (A.stats) {
    unsigned sup = n_support, cands = (unsigned)cnt;
    for (int s = 32; s > 0; s >>= 1) {
      sup += __shfl_xor((int)sup, s);
      cands += __shfl_xor((int)cands, s);
    }
    if ((threadIdx.x & 63) == 0) {
      atomicAdd(&A.stats[ENTMAX_STAT_FWD_CANDIDATES], (unsigned long long)cands);
      atomicAdd(&A.stats[ENTMAX_STAT_FWD_SUPPORT], (unsigned long long)sup);
    }
  }
}

}  // namespace entmax
