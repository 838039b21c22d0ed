// kernels_slices.hip -- matrix-core kernels whose workgroup owns 32 query rows
// (a slice: one wavefront's rows of a row group) of one head, its four
// wavefronts sharing out the slice's keys.
//
// A wavefront's unit of work is half a key tile: 32 keys.  Of the slice's
// non-empty tiles (in order), wavefront w takes the tiles of parity w / 2 and,
// of each, half w % 2.  Nothing is shared while the units are walked, so there
// is no barrier: a unit's K rows come through the wavefront's own LDS, one
// unit ahead, its V rows straight into the operand registers.  At the end the
// four partial results are combined through LDS.
//
// Operands (lane = 32 h + i): S^T = K Q^T with lane i holding key i's (A) or
// query i's (B) features in chunks of 16 bytes, halves h alternating -- any
// order of the features will do as long as both sides use the same -- and
// the scores of ONE query, keys 8 (r/4) + 4 h + r % 4, in registers r = 0..15.
// O^T += V^T P^T takes P^T straight from those registers; lane i reads
// features NB i .. NB i + NB - 1 (NB = d / 32) of the key rows the registers
// imply, whole rows per load, so output row i of block b is feature NB i + b.
#include <hip/hip_runtime.h>
#include <math.h>

#include <type_traits>

#include "bounds.hpp"
#include "launch.hpp"
#include "mfma_util.hpp"

namespace splat {
namespace {

using namespace mfma;

constexpr int kThreads = 256;            // 4 wavefronts, one slice
constexpr int kUnit = 32;                // keys per unit
constexpr int kMaxGridY = 32768;         // slices per launch dimension; more are looped over
constexpr float kRefSlack = 8.f;

typedef float f32x4_t __attribute__((ext_vector_type(4)));
typedef float f32x4u_t __attribute__((ext_vector_type(4), aligned(4)));
typedef float f32x2_t __attribute__((ext_vector_type(2)));
typedef unsigned int u32x2_t __attribute__((ext_vector_type(2)));

// ---------------------------------------------------------------- operands
template <typename T, int D>
struct Mat;

// fp32: v_mfma_f32_32x32x2_f32 (fp32 products, fp32 sums)
template <int D>
struct Mat<float, D> {
  static constexpr int NB = D / 32;
  typedef typename std::conditional<NB == 2, f32x2_t, f32x4_t>::type vrow_t;
  struct Row {               // features 8 t + 4 h .. + 3 of a Q or K row
    f32x4_t v[D / 8];
  };
  struct V {                 // features NB i .. of 8 key rows: half j of a unit
    vrow_t v[8];
  };
  static __device__ __forceinline__ f32x16_t dot(const Row& k, const Row& q) {
    f32x16_t s;
#pragma unroll
    for (int r = 0; r < 16; ++r) s[r] = 0.f;
#pragma unroll
    for (int t = 0; t < D / 8; ++t)
#pragma unroll
      for (int e = 0; e < 4; ++e)
        s = __builtin_amdgcn_mfma_f32_32x32x2f32(k.v[t][e], q.v[t][e], s, 0, 0, 0);
    return s;
  }
  static __device__ __forceinline__ void pv(f32x16_t (&o)[NB], const V& v, const float (&p)[16],
                                            int j) {
#pragma unroll
    for (int r = 0; r < 8; ++r)
#pragma unroll
      for (int b = 0; b < NB; ++b)
        o[b] = __builtin_amdgcn_mfma_f32_32x32x2f32(v.v[r][b], p[8 * j + r], o[b], 0, 0, 0);
  }
};

// bf16: v_mfma_f32_32x32x16_bf16
template <int D>
struct Mat<__bf16, D> {
  static constexpr int NB = D / 32;
  typedef typename std::conditional<NB == 2, unsigned, u32x2_t>::type vrow_t;
  struct Row {               // features 16 t + 8 h .. + 7 of a Q or K row
    bf16x8_t v[D / 16];
  };
  struct V {                 // features NB i .. of 8 key rows: half j of a unit
    vrow_t v[8];
  };
  static __device__ __forceinline__ f32x16_t dot(const Row& k, const Row& q) {
    f32x16_t s;
#pragma unroll
    for (int r = 0; r < 16; ++r) s[r] = 0.f;
#pragma unroll
    for (int t = 0; t < D / 16; ++t) s = mfma32(k.v[t], q.v[t], s);
    return s;
  }
  // block b's operand of the half's k-step: element e is key row e
  static __device__ __forceinline__ bf16x8_t vt(const V& v, int b) {
    u32x4_t a;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      unsigned x, y;
      if constexpr (NB == 2) {
        x = v.v[2 * e], y = v.v[2 * e + 1];
      } else {
        x = v.v[2 * e][b >> 1], y = v.v[2 * e + 1][b >> 1];
      }
      a[e] = __builtin_amdgcn_perm(y, x, (b & 1) ? 0x07060302u : 0x05040100u);
    }
    return __builtin_bit_cast(bf16x8_t, a);
  }
  // P as a bf16 high part plus a bf16 remainder: about 16 significant bits
  static __device__ __forceinline__ void pv(f32x16_t (&o)[NB], const V& v, const float (&p)[16],
                                            int j) {
    bf16x8_t hi, lo;
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      hi[e] = (__bf16)p[8 * j + e];
      lo[e] = (__bf16)(p[8 * j + e] - (float)hi[e]);
    }
#pragma unroll
    for (int b = 0; b < NB; ++b) {
      const bf16x8_t a = vt(v, b);
      o[b] = mfma32(a, hi, o[b]);
      o[b] = mfma32(a, lo, o[b]);
    }
  }
};

// K or Q row: 16-byte chunks 2 t + h, t < D * sizeof(T) / 32
template <typename T, int D>
__device__ __forceinline__ void load_row(typename Mat<T, D>::Row& x, const char* base,
                                         unsigned off) {
  constexpr int N = D * (int)sizeof(T) / 32;
#pragma unroll
  for (int t = 0; t < N; ++t)
    x.v[t] = *(const typename std::remove_reference<decltype(x.v[0])>::type*)(base + off + 32 * t);
}

// ------------------------------------------------------------ units of work
struct Unit {
  int kb, ks, n;       // keys kb + ks * u, u < n (n <= 32)
  int mask_block;
  int half;            // which half of the tile
  bool full;           // every key in every row of the slice
};

// Walks the slice's non-empty tiles and yields this wavefront's units.  The
// 64 lanes hold 64 tile descriptors at a time, so a unit costs no dependent
// load.
struct Units {
  const Tile* tiles;   // the group's first tile
  int nt, base, rank, lane, wave, slice;
  uint64_t left;       // non-empty tiles of the current 64 not yet visited
  int4 d;
  int mb;

  __device__ __forceinline__ void fetch() {
    d = make_int4(0, 1, 0, 0);
    mb = -1;
    if (base + lane < nt) {
      const Tile* t = tiles + base + lane;
      d = *(const int4*)t;
      mb = t->mask_block;
    }
    left = __ballot(((d.w >> (kWaveShift + 2 * slice)) & 3) != kWaveEmpty);
  }
  __device__ __forceinline__ void start(const Tile* t, int n, int lane_, int wave_, int slice_) {
    tiles = t, nt = n, base = 0, rank = 0, lane = lane_, wave = wave_, slice = slice_;
    fetch();
  }
  __device__ __forceinline__ bool next(Unit& u) {
    const int half = wave & 1;
    while (true) {
      while (left == 0) {
        base += 64;
        if (base >= nt) return false;
        fetch();
      }
      const int t = __builtin_ctzll(left);
      left &= left - 1;
      const bool mine = (rank & 1) == (wave >> 1);
      ++rank;
      const int nk = __builtin_amdgcn_readlane(d.z, t) - kUnit * half;
      if (!mine || nk <= 0) continue;
      u.ks = __builtin_amdgcn_readlane(d.y, t);
      u.kb = __builtin_amdgcn_readlane(d.x, t) + u.ks * kUnit * half;
      u.n = min(nk, kUnit);
      u.mask_block = __builtin_amdgcn_readlane(mb, t);
      u.half = half;
      const int st = (__builtin_amdgcn_readlane(d.w, t) >> (kWaveShift + 2 * slice)) & 3;
      u.full = st == kWaveFull;
      return true;
    }
  }
};

// A wavefront's view of its slice.
struct Slice {
  int lane, wave, qi, h, w;    // w: the slice's place in its group
  int row, tb, nt;
  bool row_valid;
  const uint32_t* masks;       // the slice's 32-bit mask words, two per row

  // false: the slice has no row
  __device__ __forceinline__ bool open(int s, const Group* groups, const int32_t* rows,
                                       const uint64_t* m, int L) {
    const Group grp = groups[s / kWavesPerGroup];
    w = s % kWavesPerGroup;
    if (w * kWaveRows >= grp.nrows) return false;
    lane = threadIdx.x & 63;
    wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    qi = lane & 31, h = lane >> 5;
    const int i = w * kWaveRows + qi;
    row_valid = i < grp.nrows;
    row = row_valid ? dbg::idx(rows[grp.row_off + i], L, dbg::kRow) : 0;
    tb = grp.tile_begin, nt = grp.tile_end - grp.tile_begin;
    masks = (const uint32_t*)m + 2 * i;
    return true;
  }
  // the row's membership bits in a unit
  __device__ __forceinline__ uint32_t bits(const Unit& u) const {
    return u.full ? ~0u : masks[(size_t)u.mask_block * (2 * kBM) + u.half];
  }
  __device__ __forceinline__ int key(const Unit& u, int k, int L) const {
    return dbg::idx(u.kb + u.ks * min(k, u.n - 1), L, dbg::kKey);
  }
};

// waits for this wavefront's LDS reads, and for its loads from memory
__device__ __forceinline__ void wait_lds() { asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory"); }
__device__ __forceinline__ void wait_loads() {
  asm volatile("" ::: "memory");
  __builtin_amdgcn_s_waitcnt((7 << 4) | (15 << 8));
  asm volatile("" ::: "memory");
}

// A unit's K rows go from memory into the wavefront's own LDS, 1 KB of whole
// rows per load, and from there into the operand: loaded straight into the
// operand, each load would touch 32 rows, 32 bytes of each, and K would hold
// registers a unit ahead (d = 128: 862 us against 631, full mask, L = 2048,
// 32 heads).  The 16-byte chunks of row r sit XOR-ed with r % 16 (128-byte rows:
// r / 2 % 8), so that the operand reads (16 lanes, 16 rows) are free of bank
// conflicts.  Keys past the unit's end re-read its last.
template <int CPR>
__device__ __forceinline__ int swz_row(int r) { return CPR == 8 ? (r >> 1) & 7 : r & 15; }
template <typename T, int D>
__device__ __forceinline__ void fetch_k(float* stage, const char* Kh, const Slice& s, const Unit& u,
                                        int L) {
  constexpr int RB = D * (int)sizeof(T), CPR = RB / 16, RPL = 64 / CPR;
  wait_lds();   // the unit before it has left the LDS rows that these loads fill
#pragma unroll
  for (int k = 0; k < kUnit / RPL; ++k) {
    const int r = RPL * k + s.lane / CPR;
    const int c = (s.lane % CPR) ^ swz_row<CPR>(r);
    dma16(Kh + ((unsigned)s.key(u, r, L) * (unsigned)RB + 16u * c), (char*)stage + kDmaBlock * k);
  }
}
template <typename T, int D>
__device__ __forceinline__ void load_k(typename Mat<T, D>::Row& x, const float* stage,
                                       const Slice& s) {
  constexpr int RB = D * (int)sizeof(T);
  const int off = s.qi * RB + 16 * (s.h ^ swz_row<RB / 16>(s.qi));
#pragma unroll
  for (int t = 0; t < RB / 32; ++t)
    x.v[t] = *(const typename std::remove_reference<decltype(x.v[0])>::type*)((const char*)stage +
                                                                             (off ^ (32 * t)));
}
template <typename T, int D>
__device__ __forceinline__ void load_v(typename Mat<T, D>::V& x, const char* Vh, const Slice& s,
                                       const Unit& u, int j, int L) {
  using vrow_t = typename Mat<T, D>::vrow_t;
  constexpr unsigned RB = D * sizeof(T);
  if (u.n == kUnit) {
    // whole unit: one lane offset, the rows' offsets are uniform
    const unsigned lo = (unsigned)(u.ks * 4 * s.h) * RB + (unsigned)sizeof(vrow_t) * s.qi;
#pragma unroll
    for (int r = 0; r < 8; ++r) {
      const int k = 16 * j + 8 * (r >> 2) + (r & 3);
      const char* p = Vh + (size_t)((unsigned)dbg::idx(u.kb + u.ks * k, L, dbg::kKey) * RB);
      x.v[r] = *(const vrow_t*)(p + lo);
    }
  } else {
#pragma unroll
    for (int r = 0; r < 8; ++r) {
      const int k = s.key(u, 16 * j + 8 * (r >> 2) + 4 * s.h + (r & 3), L);
      x.v[r] = *(const vrow_t*)(Vh + ((unsigned)k * RB + (unsigned)sizeof(vrow_t) * s.qi));
    }
  }
}

// f(r, present, pos) for the 16 keys of this lane: pos = the key's place
// among the row's keys of the unit
template <typename F>
__device__ __forceinline__ void for_each_key(uint32_t bits, int h, F&& f) {
  const uint32_t b = bits >> (4 * h);
  int off = h ? __builtin_popcount(bits & 0xFu) : 0;
#pragma unroll
  for (int g = 0; g < 4; ++g) {
    const uint32_t nib = (b >> (8 * g)) & 0xFu;
    const uint32_t oth = (b >> (8 * g + 4)) & 0xFu;   // the other half's next four
#pragma unroll
    for (int e = 0; e < 4; ++e)
      f(4 * g + e, (nib >> e) & 1u, off + __builtin_popcount(nib & ((1u << e) - 1u)));
    off += __builtin_popcount(nib) + __builtin_popcount(oth);
  }
}

// number of the row's columns below x.  The quotients are below 2^18 and the
// dividends below 2^24, so the float product is off by one at most.
__device__ __forceinline__ int row_count_lt(const RowRuns& rr, int x) {
  int n = 0;
#pragma unroll
  for (int r = 0; r < SPLAT_MAX_RUNS; ++r) {
    const Run q = rr.r[r];
    int c = x - q.start;
    if (q.stride != 1) {
      const int num = c + q.stride - 1;
      int f = (int)((float)num * __builtin_amdgcn_rcpf((float)q.stride));
      const int rem = num - f * q.stride;
      f += rem >= q.stride ? 1 : 0;
      f -= rem < 0 ? 1 : 0;
      c = c > 0 ? f : 0;
    }
    n += max(0, min(c, q.count));
  }
  return n;
}

// scores outside the row's runs set to -inf
__device__ __forceinline__ void mask_unit(float (&t)[16], uint32_t bits, int h) {
  const unsigned word = bits >> (4 * h);
#pragma unroll
  for (int r = 0; r < 16; ++r) t[r] = keep_if_bit(t[r], word, 8 * (r >> 2) + (r & 3));
}

// The matrix cores multiply every key row by every query's weight, 0 for the
// queries that do not have the key, and 0 * inf is NaN: with an infinity or a NaN
// in V, rows that lack the key turn NaN as well.  z turns NaN when V holds one in
// half a unit in which some row lacks some key; the lane's row is then marked by
// a NaN, and combine forms such rows again one by one (in the chain all of the
// slice's).  (combine would find them without z, but the fused loop without the
// check is scheduled worse: window 256 + 32 global, L = 2048, 12 heads 59 -> 73 us.)
// With bf16 V no such check is made: there a row may see the keys of its tile.
template <typename T, int D>
__device__ __forceinline__ void check_v(float& z, const typename Mat<T, D>::V& v, const Unit& u) {
  if constexpr (std::is_same<T, float>::value) {
    if (!u.full) {
#pragma unroll
      for (int r = 0; r < 8; ++r)
#pragma unroll
        for (int b = 0; b < D / 32; ++b) z = fmaf(v.v[r][b], 0.f, z);
    }
  }
}

// --------------------------------------------------------- combining, output
// LDS of a slice kernel: each wavefront's partial O (its staging area before
// that), the row references and sums.
template <int D>
struct Shared {
  static constexpr int OS = D + 4;                 // floats per staged O row
  float o[kWavesPerGroup][kWaveRows * OS];
  float m[kWavesPerGroup][kWaveRows];
  float l[kWavesPerGroup][kWaveRows];
  int redo;                                        // the chain: some V value is not finite
};

template <typename OutT>
__device__ __forceinline__ void store_o4(OutT* p, f32x4_t v) {
  store4<OutT>(p, v[0], v[1], v[2], v[3]);
}

// Sum of the wavefronts' O^T, times inv(row i), written as whole rows: every
// thread sums four features of one row at a time, eight lanes along a row.
// CHECK: a row whose result is not finite is not stored (O may lie over Q) but
// formed by again(row): by its keys one after the other.  That order of the sums
// may stay within fp32's range where this one does not, and the row code keeps the
// fused kernel's weights at 1 and below, which reach 2^kRefSlack before the
// division by their sum here.  Each wavefront looks after the eight rows it sums.
template <int D, bool CHECK, typename OutT, typename F, typename G>
__device__ __forceinline__ void combine(Shared<D>& sh, const f32x16_t (&o)[D / 32], const Slice& s,
                                        OutT* Oh, F&& inv, G&& again) {
  constexpr int NB = D / 32, OS = Shared<D>::OS;
  float* const mine = sh.o[s.wave] + s.qi * OS;
#pragma unroll
  for (int g = 0; g < 4; ++g)
#pragma unroll
    for (int c = 0; c < NB; ++c) {      // features NB (8 g + 4 h) + 4 c .. + 3
      f32x4_t v;
#pragma unroll
      for (int e = 0; e < 4; ++e) v[e] = o[(4 * c + e) % NB][4 * g + (4 * c + e) / NB];
      *(f32x4_t*)(mine + NB * (8 * g + 4 * s.h) + 4 * c) = v;
    }
  __syncthreads();
  const int r = threadIdx.x >> 3;                  // row of the slice
  const int lane_r = (int)__shfl(s.row_valid ? s.row : -1, r & 31, 64);
  f32x4_t v[NB];
  float z = 0.f;
  if (lane_r >= 0) {
    const float f = inv(r, lane_r);
#pragma unroll
    for (int k = 0; k < NB; ++k) {
      const int c = 4 * (threadIdx.x & 7) + 32 * k;
      v[k] = *(const f32x4_t*)(sh.o[0] + r * OS + c);
#pragma unroll
      for (int w = 1; w < kWavesPerGroup; ++w) v[k] += *(const f32x4_t*)(sh.o[w] + r * OS + c);
      v[k] *= f;
      if (CHECK)
#pragma unroll
        for (int e = 0; e < 4; ++e) z = fmaf(v[k][e], 0.f, z);
    }
  }
  const uint64_t bad = CHECK ? __ballot(z != z) : 0;
  if (lane_r >= 0 && ((bad >> (s.lane & 56)) & 0xffu) == 0) {
    OutT* const orow = Oh + (size_t)lane_r * D;
#pragma unroll
    for (int k = 0; k < NB; ++k) store_o4<OutT>(orow + 4 * (threadIdx.x & 7) + 32 * k, v[k]);
  }
  if (CHECK && bad != 0)
    for (int k = 0; k < 64; k += 8)
      if ((bad >> k) & 0xffu) again(__builtin_amdgcn_readlane(lane_r, k));
}

// exp(x - m) as the row softmax forms it
__device__ __forceinline__ float exp_from(float x, float m) {
  return exp2_hw((x - m) * 1.4426950408889634f);
}
// the factor that takes a sum from reference m to mt >= m (-inf: nothing summed)
__device__ __forceinline__ float rescale(float m, float mt) {
  return m == -INFINITY ? 0.f : exp_from(m, mt);
}

// ---------------------------------------------------------- one row, VALU
// column of the k-th value of a row (k < row nnz)
__device__ __forceinline__ int col_of(const RowRuns& rr, int k) {
  int j = 0;
#pragma unroll
  for (int r = 0; r < SPLAT_MAX_RUNS; ++r) {
    const Run q = rr.r[r];
    if (k >= q.prefix && k < q.prefix + q.count) j = q.start + q.stride * (k - q.prefix);
  }
  return j;
}

__device__ __forceinline__ void store1(float* p, float v) { *p = v; }
__device__ __forceinline__ void store1(__bf16* p, float v) { *p = (__bf16)v; }

// The fused forward of row i by one wavefront: scores by lanes over 64 keys at
// a time, O by lanes over the features; only the row's own keys are read.
template <int D, typename OutT>
__device__ __forceinline__ void fused_row(int i, int lane, const RowRuns* runs,
                                          const int32_t* row_ptr, int L, const float* Qh,
                                          const float* Kh, const float* Vh, float scale,
                                          OutT* Oh) {
  constexpr int NC = D / 64;
  const RowRuns rr = runs[i];
  const int n = row_ptr[i + 1] - row_ptr[i];
  const float* const q = Qh + (size_t)i * D;
  // m: the largest score so far, from the lowest float on: against that a score
  // of -inf weighs 0 (against -inf itself NaN).  O of a row without keys is 0 / 1,
  // of one whose keys all score -inf 0 / 0.
  float m = -__FLT_MAX__, l = n > 0 ? 0.f : 1.f, acc[NC];
#pragma unroll
  for (int b = 0; b < NC; ++b) acc[b] = 0.f;
#pragma unroll 1
  for (int k0 = 0; k0 < n; k0 += 64) {
    const bool valid = k0 + lane < n;
    int j = 0;
    float x = -INFINITY;
    if (valid) {
      j = dbg::idx(col_of(rr, k0 + lane), L, dbg::kKey);
      const float* const k = Kh + (size_t)j * D;
      float d[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int c = 0; c < D; c += 4) {
        const f32x4_t kv = *(const f32x4_t*)(k + c);
#pragma unroll
        for (int e = 0; e < 4; ++e) d[e] = fmaf(q[c + e], kv[e], d[e]);
      }
      x = ((d[0] + d[1]) + (d[2] + d[3])) * scale;
    }
    const float mn = fmaxf(m, wave_max(x));
    const float alpha = expf(m - mn);
    const float p = valid ? expf(x - mn) : 0.f;
    l = l * alpha + wave_sum(p);
#pragma unroll
    for (int b = 0; b < NC; ++b) acc[b] *= alpha;
    auto key = [&](int t) {
      const float pt = __builtin_bit_cast(
          float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, p), t));
      const float* const v = Vh + (size_t)__builtin_amdgcn_readlane(j, t) * D;
#pragma unroll
      for (int b = 0; b < NC; ++b) acc[b] = fmaf(pt, v[64 * b + lane], acc[b]);
    };
    const int cnt = min(64, n - k0);
    int t = 0;
#pragma unroll 1
    for (; t + 8 <= cnt; t += 8)
#pragma unroll
      for (int e = 0; e < 8; ++e) key(t + e);
#pragma unroll 1
    for (; t < cnt; ++t) key(t);
    m = mn;
  }
  const float inv = 1.f / l;
#pragma unroll
  for (int b = 0; b < NC; ++b) store1(Oh + (size_t)i * D + 64 * b + lane, acc[b] * inv);
}

// One wavefront per row: the launches too small for the slices below.
template <int D, typename OutT>
__global__ __launch_bounds__(kThreads) void k_fused_rows(
    const int32_t* __restrict__ row_ptr, const RowRuns* __restrict__ runs, int L,
    const float* __restrict__ Q, const float* __restrict__ K, const float* __restrict__ V,
    float scale, OutT* __restrict__ O) {
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int i = blockIdx.y * 4 + wave;
  if (i >= L) return;
  const size_t head = (size_t)blockIdx.x * L * D;
  fused_row<D, OutT>(i, threadIdx.x & 63, runs, row_ptr, L, Q + head, K + head, V + head, scale,
                     O + head);
}

// ------------------------------------------------------------- fused forward
// O = softmax_nz(scale * M (x) Q K^T) V, the online softmax per wavefront over
// its units, the four (reference, sum, O) combined at the end.  A row takes its
// first unit's maximum as its reference and keeps it while later maxima stay
// within 2^kRefSlack of it: p then lies in [0, 2^kRefSlack], in fp32 as exact
// as below 1, and few units rescale O.  (Rows whose O leaves fp32's range for it
// are formed again, see combine.)
//
// fp32 is bound by the matrix cores: a unit is 64 (d = 64) v_mfma_f32_32x32x2
// of 64 cycles.  Full mask, L = 2048, 64 heads, d = 64: 651 us, 106 TFLOP/s of
// the 153 that a large fp32 matrix product reaches (without the loads of K and
// V 127); a wavefront per row (lanes' own dot products) ran at 7 TFLOP/s.
// Window 256 + 32 global, L = 2048, 12 heads: 620 -> 59 us; there the slice of
// the global rows, 16 units per wavefront, is the longest chain.  Two
// wavefronts per SIMD; three (168 registers, some spilled) took 86 us against
// 63, and the next unit's products beside this one's softmax 65 against 60.
template <int D, typename OutT>
__global__ __launch_bounds__(kThreads, 2) void k_fused_slices(
    const Group* __restrict__ groups, const int32_t* __restrict__ rows,
    const int32_t* __restrict__ row_ptr, const RowRuns* __restrict__ runs,
    const Tile* __restrict__ tiles, const uint64_t* __restrict__ masks, int L, int n_slices,
    const float* __restrict__ Q, const float* __restrict__ K, const float* __restrict__ V,
    float scale, OutT* __restrict__ O) {
  using T = float;
  using M = Mat<T, D>;
  constexpr int NB = D / 32;
  __shared__ __attribute__((aligned(16))) Shared<D> sh;
  const size_t head = (size_t)blockIdx.x * L * D;
  const char* Kh = (const char*)(K + head);
  const char* Vh = (const char*)(V + head);
  // sl2 = scale * log2(e) > 0: the sign of a negative scale, and a zero one, go to Q
  const float sl2 = scale == 0.f ? 1.f : fabsf(scale) * 1.4426950408889634f;
  const float sgn = scale == 0.f ? 0.f : copysignf(1.f, scale);
  for (int sl = blockIdx.y; sl < n_slices; sl += gridDim.y) {
    Slice s;
    if (!s.open(sl, groups, rows, masks, L)) continue;
    typename M::Row q;
    load_row<T, D>(q, (const char*)(Q + head),
                   (unsigned)s.row * (D * (unsigned)sizeof(T)) + 16u * s.h);
    for (auto& x : q.v) x *= sgn;
    f32x16_t o[NB];
#pragma unroll
    for (int b = 0; b < NB; ++b)
#pragma unroll
      for (int r = 0; r < 16; ++r) o[b][r] = 0.f;
    // the row's reference (log2 domain) and the sum of this half's keys
    float m = -INFINITY, l = 0.f;
    float z = 0.f;

    float* const stage = sh.o[s.wave];
    Units it;
    it.start(tiles + s.tb, s.nt, s.lane, s.wave, s.w);
    Unit u;
    bool more = it.next(u);
    if (more) fetch_k<T, D>(stage, Kh, s, u, L);
    while (more) {
      // d = 128: V is loaded where no K is held, half a unit at a time, for two
      // wavefronts per SIMD (256 registers, and 22 spilled: 92 bytes a lane)
      wait_loads();
      typename M::Row k;
      load_k<T, D>(k, stage, s);
      typename M::V v0, v1;
      if (D == 64) load_v<T, D>(v0, Vh, s, u, 0, L);
      const uint32_t bits = s.bits(u);
      const f32x16_t acc = M::dot(k, q);
      if (D != 64) {
        __builtin_amdgcn_sched_barrier(0);
        load_v<T, D>(v0, Vh, s, u, 0, L);
      }
      Unit nu;
      const bool next = it.next(nu);
      if (next) fetch_k<T, D>(stage, Kh, s, nu, L);
      float p[16];
#pragma unroll
      for (int r = 0; r < 16; ++r) p[r] = acc[r];
      if (!u.full) mask_unit(p, bits, s.h);
      float mx0 = p[0], mx1 = p[8];
#pragma unroll
      for (int r = 1; r < 8; ++r) {
        mx0 = fmaxf(mx0, p[r]);
        mx1 = fmaxf(mx1, p[8 + r]);
      }
      float mx = fmaxf(mx0, mx1);
      mx = fmaxf(mx, lane_xor32(mx)) * sl2;
      if (__any(mx > m + kRefSlack)) {
        const float mn = mx > m + kRefSlack ? mx : m;
        const float alpha = m == -INFINITY ? 0.f : exp2_hw(m - mn);
        l *= alpha;
#pragma unroll
        for (int b = 0; b < NB; ++b)
#pragma unroll
          for (int r = 0; r < 16; ++r) o[b][r] *= alpha;
        m = mn;
      }
      const float mu = m == -INFINITY ? 0.f : m;   // no key yet: exp2(-inf - 0) = 0
      float l0 = 0.f, l1 = 0.f;
#pragma unroll
      for (int r = 0; r < 16; r += 2) {
        p[r] = exp2_hw(fmaf(p[r], sl2, -mu)), p[r + 1] = exp2_hw(fmaf(p[r + 1], sl2, -mu));
        l0 += p[r], l1 += p[r + 1];
      }
      l += l0 + l1;
      if (D == 64) load_v<T, D>(v1, Vh, s, u, 1, L);
      check_v<T, D>(z, v0, u);
      M::pv(o, v0, p, 0);
      if (D != 64) {
        __builtin_amdgcn_sched_barrier(0);
        load_v<T, D>(v1, Vh, s, u, 1, L);
      }
      check_v<T, D>(z, v1, u);
      M::pv(o, v1, p, 1);
      u = nu, more = next;
    }

    l += lane_xor32(l);
    if (s.h == 0) sh.m[s.wave][s.qi] = m, sh.l[s.wave][s.qi] = l;
    __syncthreads();
    // row i's reference over the wavefronts, and a wavefront's factor to it
    auto top = [&](int i) {
      return fmaxf(fmaxf(sh.m[0][i], sh.m[1][i]), fmaxf(sh.m[2][i], sh.m[3][i]));
    };
    auto factor = [&](float mw, float mt) { return mw == -INFINITY ? 0.f : exp2_hw(mw - mt); };
    const float f = factor(m, top(s.qi));
#pragma unroll
    for (int b = 0; b < NB; ++b)
#pragma unroll
      for (int r = 0; r < 16; ++r) o[b][r] *= f;
    if (z != z) o[0][0] = z;
    auto inv = [&](int i, int row) {
      const float mt = top(i);
      float lt = 0.f;
#pragma unroll
      for (int w = 0; w < kWavesPerGroup; ++w) lt += sh.l[w][i] * factor(sh.m[w][i], mt);
      if (lt > 0.f) return 1.f / lt;
      // no key: 0; a NaN is in O already; keys that all score -inf: NaN
      return lt == 0.f && row_ptr[row] != row_ptr[row + 1] ? NAN : 0.f;
    };
    combine<D, true, OutT>(sh, o, s, O + head, inv, [&](int i) {
      fused_row<D, OutT>(i, s.lane, runs, row_ptr, L, Q + head, K + head, V + head, scale, O + head);
    });
    __syncthreads();   // LDS is reused by the next slice
  }
}

// ------------------------------------------------------------ values in ACSR
// Where the values of a row's keys of a unit sit: position `pos` of head bh
// on, its present keys in order.
__device__ __forceinline__ int unit_pos(const RowRuns& rr, int row_begin, const Unit& u) {
  return row_begin + row_count_lt(rr, u.kb);
}

// The unit's values of every row to memory.  Each row's present keys are
// gathered in LDS and leave as row segments, eight lanes of 16 bytes a row
// (straight from the registers a store would touch 32 rows, 32 bytes each).
__device__ __forceinline__ void write_values(float* dst, int64_t nnz, const float (&x)[16],
                                             uint32_t bits, const Unit& u, int pos,
                                             const Slice& s, float* stage) {
  // value k of row r: its 16-byte chunk k / 4 XOR-ed with r % 8 (bank conflicts)
  auto at = [&](int r, int k) { return stage + r * kUnit + 4 * ((k >> 2) ^ (r & 7)) + (k & 3); };
  if (u.full) {
#pragma unroll
    for (int g = 0; g < 4; ++g)
      *(f32x4_t*)at(s.qi, 8 * g + 4 * s.h) =
          f32x4_t{x[4 * g], x[4 * g + 1], x[4 * g + 2], x[4 * g + 3]};
  } else {
    for_each_key(bits, s.h, [&](int r, unsigned present, int k) {
      if (present) *at(s.qi, k) = x[r];
    });
  }
  const int n = s.row_valid ? __builtin_popcount(bits) : 0;
  const int c = 4 * (s.lane & 7);
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    const int r = 8 * k + (s.lane >> 3);
    const int nr = __shfl(n, r, 64), pr = __shfl(pos, r, 64);
    if (c >= nr) continue;
    const f32x4_t v = *(const f32x4_t*)at(r, c);
    float* const p = dst + pr;
    if (c + 4 <= nr) {
      *(f32x4u_t*)(p + dbg::rel(c, (int64_t)pr, nnz - 3, dbg::kValue)) = v;
    } else {
#pragma unroll
      for (int e = 0; e < 3; ++e)
        if (c + e < nr) p[dbg::rel(c + e, (int64_t)pr, nnz, dbg::kValue)] = v[e];
    }
  }
}

// f(r, place) for the keys of this lane that its row has: the value's place in
// the head's column-major values.  Lane i reads key i's descriptor; where every
// column steps by one row, as in all but dilated masks, a value's place is
// (ptr - start) + row.  The column-wise analysis ends at 2^28 values a head, so
// places times four fit 32 bits.
template <typename F>
__device__ __forceinline__ void for_each_place(uint32_t bits, int64_t nnz, const Unit& u,
                                               const ColRun* cols, const Slice& s, int L,
                                               float* stage, F&& f) {
  const ColRun mine = cols[s.key(u, s.qi, L)];
  const uint32_t b = bits >> (4 * s.h);
  if (__all(mine.stride == 1)) {
    int* const base = (int*)stage;
    base[s.qi] = mine.ptr - mine.start;
    wait_lds();
#pragma unroll
    for (int g = 0; g < 4; ++g) {
      const int4 c = *(const int4*)(base + 8 * g + 4 * s.h);
#pragma unroll
      for (int e = 0; e < 4; ++e)
        if ((b >> (8 * g + e)) & 1u)
          f(4 * g + e, dbg::idx((&c.x)[e] + s.row, (int)nnz, dbg::kColPos));
    }
    wait_lds();
    return;
  }
#pragma unroll
  for (int r = 0; r < 16; ++r) {
    const int k = 8 * (r >> 2) + (r & 3);
    const ColRun c = cols[s.key(u, k + 4 * s.h, L)];
    if ((b >> k) & 1u) f(r, dbg::idx(col_pos(c, s.row), (int)nnz, dbg::kColPos));
  }
}

// ---------------------------------------------------------------- R-SDDMM
// fp32: 32 MFMAs (d = 64) a unit against 4 KB of scores written; measured per
// launch, a wavefront per row against this: strided+local 128, L = 2048, 12
// heads 101 -> 21.5 us; dilated 3, L = 1000, d = 128, 8 heads 83 -> 22.3.
// LDS: K and the staged values, at d = 128 exactly half a CU's 160 KB.
template <typename T, int D>
__global__ __launch_bounds__(kThreads, D == 64 ? 3 : 2) void k_rsddmm_slices(
    const Group* __restrict__ groups, const int32_t* __restrict__ rows,
    const int32_t* __restrict__ row_ptr, const RowRuns* __restrict__ runs,
    const Tile* __restrict__ tiles, const uint64_t* __restrict__ masks, int L, int64_t nnz,
    int n_slices, const T* __restrict__ Q, const T* __restrict__ K, float scale,
    float* __restrict__ S) {
  using M = Mat<T, D>;
  __shared__ __attribute__((aligned(16))) float kst[kWavesPerGroup][kUnit * D * sizeof(T) / 4];
  __shared__ __attribute__((aligned(16))) float vst[kWavesPerGroup][kWaveRows * kUnit];
  const size_t head = (size_t)blockIdx.x * L * D;
  const char* Kh = (const char*)(K + head);
  float* const Sh = S + (size_t)blockIdx.x * nnz;
  for (int sl = blockIdx.y; sl < n_slices; sl += gridDim.y) {
    Slice s;
    if (!s.open(sl, groups, rows, masks, L)) continue;
    typename M::Row q;
    load_row<T, D>(q, (const char*)(Q + head),
                   (unsigned)s.row * (D * (unsigned)sizeof(T)) + 16u * s.h);
    const RowRuns rr = runs[s.row];
    const int row_begin = row_ptr[s.row];
    Units it;
    it.start(tiles + s.tb, s.nt, s.lane, s.wave, s.w);
    Unit u;
    bool more = it.next(u);
    if (more) fetch_k<T, D>(kst[s.wave], Kh, s, u, L);
    while (more) {
      wait_loads();
      typename M::Row k;
      load_k<T, D>(k, kst[s.wave], s);
      const uint32_t bits = s.bits(u);
      const f32x16_t acc = M::dot(k, q);
      Unit nu;
      const bool next = it.next(nu);
      if (next) fetch_k<T, D>(kst[s.wave], Kh, s, nu, L);
      float x[16];
#pragma unroll
      for (int r = 0; r < 16; ++r) x[r] = acc[r] * scale;
      write_values(Sh, nnz, x, bits, u, unit_pos(rr, row_begin, u), s, vst[s.wave]);
      u = nu, more = next;
    }
  }
}

// The scores of a row by one wavefront, a key per lane.
template <int D>
__global__ __launch_bounds__(64) void k_rsddmm_rows(
    const int32_t* __restrict__ row_ptr, const RowRuns* __restrict__ runs, int L, int64_t nnz,
    const float* __restrict__ Q, const float* __restrict__ K, float scale,
    float* __restrict__ S) {
  const int i = blockIdx.x, bh = blockIdx.y, lane = threadIdx.x;
  __shared__ float qs[D];
  const size_t head = (size_t)bh * L * D;
  for (int c = lane; c < D; c += 64) qs[c] = Q[head + (size_t)i * D + c];
  __syncthreads();
  const RowRuns rr = runs[i];
  const int64_t r0 = row_ptr[i];
  float* const out = S + (size_t)bh * nnz + r0;
#pragma unroll
  for (int r = 0; r < SPLAT_MAX_RUNS; ++r) {
    const Run q = rr.r[r];
    for (int k = lane; k < q.count; k += 64) {
      const int j = dbg::idx(q.start + q.stride * k, L, dbg::kKey);
      const float* const key = K + head + (size_t)j * D;
      float x = 0.f;
#pragma unroll 8   // eight 16-byte loads in flight (all sixteen of d = 64: 2.9 us for 2.6)
      for (int c = 0; c < D; c += 4)
#pragma unroll
        for (int e = 0; e < 4; ++e) x = fmaf(qs[c + e], key[c + e], x);
      out[dbg::rel(q.prefix + k, r0, nnz, dbg::kValue)] = x * scale;
    }
  }
}

// ----------------------------------------------------------------- R-SpMM
// COL: P holds the head's values in column-major order, value (i, j) at
// col_pos(cols[j], i).  fp32, a wavefront per row against slices: strided+local
// 128, L = 2048, 12 heads 54 -> 20.6 us; dilated 3, L = 1000, d = 128, 8 heads
// 64 -> 20.6, and with the walk advanced after V's loads, which ended the
// spills, 22.1 -> 19.1 under a kernel trace; per unit 32 MFMAs (d = 64) and V's
// 8 KB against P's 4 KB.

// O of row i by one wavefront, lanes over the features.
template <int D, typename OutT, bool COL>
__device__ __forceinline__ void spmm_row(int i, int lane, const RowRuns* runs,
                                         const int32_t* row_ptr, const ColRun* cols, int L,
                                         int64_t nnz, const float* Ph, const float* Vh, OutT* Oh) {
  constexpr int NC = D / 64;
  const RowRuns rr = runs[i];
  const int64_t r0 = COL ? 0 : row_ptr[i];   // p's position in the head
  const float* const p = Ph + r0;
  float acc[NC];
#pragma unroll
  for (int b = 0; b < NC; ++b) acc[b] = 0.f;
#pragma unroll
  for (int r = 0; r < SPLAT_MAX_RUNS; ++r) {
    const Run q = rr.r[r];
    auto key = [&](int k) {
      const int j = dbg::idx(q.start + q.stride * k, L, dbg::kKey);
      const float pk = COL ? p[dbg::idx((int64_t)col_pos(cols[j], i), nnz, dbg::kColPos)]
                           : p[dbg::rel(q.prefix + k, r0, nnz, dbg::kValue)];
      const float* const v = Vh + (size_t)j * D;
#pragma unroll
      for (int b = 0; b < NC; ++b) acc[b] = fmaf(pk, v[64 * b + lane], acc[b]);
    };
    int k = 0;   // eight loads in flight (four: up to 1.3 times longer on long rows)
#pragma unroll 1
    for (; k + 8 <= q.count; k += 8)
#pragma unroll
      for (int e = 0; e < 8; ++e) key(k + e);
    if (k + 4 <= q.count) {
#pragma unroll
      for (int e = 0; e < 4; ++e) key(k + e);
      k += 4;
    }
#pragma unroll 1
    for (; k < q.count; ++k) key(k);
  }
#pragma unroll
  for (int b = 0; b < NC; ++b) store1(Oh + (size_t)i * D + 64 * b + lane, acc[b]);
}

template <int D, typename OutT, bool COL>
__global__ __launch_bounds__(64) void k_rspmm_rows(
    const int32_t* __restrict__ row_ptr, const RowRuns* __restrict__ runs,
    const ColRun* __restrict__ cols, int L, int64_t nnz, const float* __restrict__ P,
    const float* __restrict__ V, OutT* __restrict__ O) {
  const size_t head = (size_t)blockIdx.y * L * D;
  spmm_row<D, OutT, COL>(blockIdx.x, threadIdx.x, runs, row_ptr, cols, L, nnz,
                         P + (size_t)blockIdx.y * nnz, V + head, O + head);
}

template <typename T, int D, typename OutT, bool COL>
__global__ __launch_bounds__(kThreads, D == 64 ? 3 : 2) void k_rspmm_slices(
    const Group* __restrict__ groups, const int32_t* __restrict__ rows,
    const int32_t* __restrict__ row_ptr, const RowRuns* __restrict__ runs,
    const Tile* __restrict__ tiles, const uint64_t* __restrict__ masks,
    const ColRun* __restrict__ cols, int L, int64_t nnz, int n_slices,
    const float* __restrict__ P, const T* __restrict__ V, OutT* __restrict__ O) {
  using M = Mat<T, D>;
  // bf16: P is read a unit ahead, beside the products of the unit before (three
  // steps, window 512 + 64 global, 16 heads 273.0 -> 271.7 us).  fp32 is bound by
  // its products and d = 128 by registers: ahead 45.8 us against 44.7 (three
  // steps, dilated 3, L = 1000, d = 128, 8 heads).
  constexpr bool kAhead = sizeof(T) == 2, kF32 = !kAhead;
  constexpr int NB = D / 32;
  __shared__ __attribute__((aligned(16))) Shared<D> sh;
  const size_t head = (size_t)blockIdx.x * L * D;
  const char* Vh = (const char*)(V + head);
  const float* const Ph = P + (size_t)blockIdx.x * nnz;
  for (int sl = blockIdx.y; sl < n_slices; sl += gridDim.y) {
    Slice s;
    if (!s.open(sl, groups, rows, masks, L)) continue;
    RowRuns rr;
    if (!COL) rr = runs[s.row];
    const int row_begin = row_ptr[s.row];
    f32x16_t o[NB];
#pragma unroll
    for (int b = 0; b < NB; ++b)
#pragma unroll
      for (int r = 0; r < 16; ++r) o[b][r] = 0.f;
    float z = 0.f;
    // the unit's values of this lane's row, 0 where the row lacks the key
    auto load_p = [&](float(&p)[16], const Unit& u) {
      const uint32_t bits = s.row_valid ? s.bits(u) : 0u;
      if (COL) {
#pragma unroll
        for (int r = 0; r < 16; ++r) p[r] = 0.f;
        for_each_place(bits, nnz, u, cols, s, L, sh.o[s.wave], [&](int r, int at) {
          p[r] = *(const float*)((const char*)Ph + 4u * (unsigned)at);
        });
        return;
      }
      const int pos = unit_pos(rr, row_begin, u);
      const float* src = Ph + pos;
      if (u.full && s.row_valid) {
#pragma unroll
        for (int g = 0; g < 4; ++g) {
          const f32x4u_t a = *(const f32x4u_t*)(src + dbg::rel(8 * g + 4 * s.h, (int64_t)pos,
                                                               nnz - 3, dbg::kValue));
#pragma unroll
          for (int e = 0; e < 4; ++e) p[4 * g + e] = a[e];
        }
      } else {
        for_each_key(bits, s.h, [&](int r, unsigned present, int k) {
          p[r] = present ? src[dbg::rel(k, (int64_t)pos, nnz, dbg::kValue)] : 0.f;
        });
      }
    };
    Units it;
    it.start(tiles + s.tb, s.nt, s.lane, s.wave, s.w);
    Unit u, nu;
    bool more = it.next(u);
    float p[16];
    if (kAhead && more) load_p(p, u);
    while (more) {
      typename M::V v0, v1;
      load_v<T, D>(v0, Vh, s, u, 0, L);
      load_v<T, D>(v1, Vh, s, u, 1, L);
      const bool next = it.next(nu);
      float pn[16];
      if (!kAhead) load_p(p, u);
      if (kAhead && next) load_p(pn, nu);
      check_v<T, D>(z, v0, u);
      M::pv(o, v0, p, 0);
      check_v<T, D>(z, v1, u);
      M::pv(o, v1, p, 1);
      if (kAhead)
#pragma unroll
        for (int r = 0; r < 16; ++r) p[r] = pn[r];
      u = nu, more = next;
    }
    if (z != z) o[0][0] = z;
    combine<D, kF32, OutT>(
        sh, o, s, O + head, [](int, int) { return 1.f; },
        [&](int i) {
          if constexpr (kF32)
            spmm_row<D, OutT, COL>(i, s.lane, runs, row_ptr, cols, L, nnz, Ph, V + head, O + head);
        });
    __syncthreads();   // LDS is reused by the next slice
  }
}

// ------------------------------------------------------- the unfused chain
// P = softmax_nz(scale * M (x) Q K^T) and O = P V in one kernel: P is written
// once and never read back.  Pass 1 forms each row's maximum and sum over its
// units (per lane; halves and wavefronts combined at the end), pass 2 forms the
// scores again -- the first unit's are kept -- and from them P and O.  The
// values are those of the single steps: fp32 scores, the exact maximum, P in
// fp32; with bf16 V the products take P as a bf16 high part plus a remainder.
// OUT: 0 = O alone, 1 = O and P, 2 = O, P and the column-major copy Pt.
//
// Bound by the stores of P at large sizes (window 512 + 64 global, L = 4096, 64
// heads, 1.1 GB of P: 569 us against 1006 for three launches that store S, read
// it, store P and read it), by the dependent loads of one slice at small ones
// (blocked 64, L = 1024, 16 heads: 7.1 us with O alone, 9.9 with P, 26.5 for
// three launches).  Window 128, L = 1024, 64 heads, while the buffers fit the
// caches: 45 us with P, 57 with Pt as well (134 for four launches); over new inputs
// from call to call 80 with Pt.  Registers: three wavefronts per SIMD at bf16, d =
// 64 (two: 53 us against 45 with P, window 128), with 2 registers spilled with P,
// 10 with Pt; two at bf16, d = 128 (three: 159 us against 101, dilated 2, L = 4096)
// and at fp32, d = 64.  At fp32, d = 128 the values wait apart from K, 87 KB of LDS
// in all: one workgroup a CU, one wavefront per SIMD.
template <typename T, int D, typename OutT, int OUT>
__global__ __launch_bounds__(kThreads, D == 64 && sizeof(T) == 2 ? 3 : 2) void k_chain_slices(
    const Group* __restrict__ groups, const int32_t* __restrict__ rows,
    const int32_t* __restrict__ row_ptr, const RowRuns* __restrict__ runs,
    const Tile* __restrict__ tiles, const uint64_t* __restrict__ masks,
    const ColRun* __restrict__ cols, int L, int64_t nnz, int n_slices, const T* __restrict__ Q,
    const T* __restrict__ K, const T* __restrict__ V, float scale, float* P, float* Pt,
    OutT* __restrict__ O) {
  using M = Mat<T, D>;
  constexpr bool kF32 = std::is_same<T, float>::value;
  constexpr int NB = D / 32;
  constexpr int KF = kUnit * D * (int)sizeof(T) / 4;   // floats of a staged K unit
  __shared__ __attribute__((aligned(16))) Shared<D> sh;
  // values on their way to P: beside K in the wavefront's part of sh.o where
  // both fit (bf16), apart from it otherwise
  constexpr bool kApart = KF + kWaveRows * kUnit > kWaveRows * Shared<D>::OS;
  __shared__ __attribute__((aligned(16))) float apart[kApart ? kWavesPerGroup : 1]
                                                     [kApart ? kWaveRows * kUnit : 4];
  __shared__ RowRuns rrs[OUT ? kWaveRows : 1];
  const size_t head = (size_t)blockIdx.x * L * D;
  const char* Kh = (const char*)(K + head);
  const char* Vh = (const char*)(V + head);
  float* const Ph = P + (size_t)blockIdx.x * nnz;
  for (int sl = blockIdx.y; sl < n_slices; sl += gridDim.y) {
    Slice s;
    if (!s.open(sl, groups, rows, masks, L)) continue;
    float* const kst = sh.o[s.wave];
    float* const vst = kApart ? apart[s.wave] : kst + KF;
    typename M::Row q, k;
    load_row<T, D>(q, (const char*)(Q + head),
                   (unsigned)s.row * (D * (unsigned)sizeof(T)) + 16u * s.h);
    // the rows' runs wait in LDS: they would hold 16 registers a lane
    int row_begin = 0;
    if (OUT) {
      row_begin = row_ptr[s.row];
      if (threadIdx.x < kWaveRows) rrs[s.qi] = runs[s.row];
    }
    if (threadIdx.x == 0) sh.redo = 0;

    Units it;
    Unit u, nu;
    it.start(tiles + s.tb, s.nt, s.lane, s.wave, s.w);
    bool more = it.next(u), kept = false;
    if (more) fetch_k<T, D>(kst, Kh, s, u, L);
    f32x16_t acc0;
    float m = -INFINITY, l = 0.f;
    while (more) {
      const uint32_t bits = s.bits(u);
      wait_loads();
      load_k<T, D>(k, kst, s);
      const f32x16_t acc = M::dot(k, q);
      if (!kept) acc0 = acc, kept = true;
      const bool next = it.next(nu);
      if (next) fetch_k<T, D>(kst, Kh, s, nu, L);
      float x[16];
#pragma unroll
      for (int r = 0; r < 16; ++r) x[r] = acc[r] * scale;
      if (!u.full) mask_unit(x, bits, s.h);
      float mx = m;
#pragma unroll
      for (int r = 0; r < 16; ++r) mx = fmaxf(mx, x[r]);
      const float mu = mx == -INFINITY ? 0.f : mx;   // no key yet: exp(-inf - 0) = 0
      l *= m == -INFINITY ? 0.f : exp_from(m, mu);
      m = mx;
      float l0 = 0.f, l1 = 0.f;
#pragma unroll
      for (int r = 0; r < 16; r += 2) l0 += exp_from(x[r], mu), l1 += exp_from(x[r + 1], mu);
      l += l0 + l1;
      u = nu, more = next;
    }
    {
      const float mo = lane_xor32(m), lo = lane_xor32(l), mt = fmaxf(m, mo);
      l = l * rescale(m, mt) + lo * rescale(mo, mt);
      m = mt;
    }
    if (s.h == 0) sh.m[s.wave][s.qi] = m, sh.l[s.wave][s.qi] = l;
    // the second pass's first units, under the barrier
    it.start(tiles + s.tb, s.nt, s.lane, s.wave, s.w);
    more = it.next(u);
    bool next = more && it.next(nu);
    if (next) fetch_k<T, D>(kst, Kh, s, nu, L);
    __syncthreads();
    float mt = -INFINITY, lt = 0.f;
#pragma unroll
    for (int w = 0; w < kWavesPerGroup; ++w) mt = fmaxf(mt, sh.m[w][s.qi]);
#pragma unroll
    for (int w = 0; w < kWavesPerGroup; ++w) lt += sh.l[w][s.qi] * rescale(sh.m[w][s.qi], mt);
    const float mu = mt == -INFINITY ? 0.f : mt, inv = 1.f / lt;

    f32x16_t o[NB];
#pragma unroll
    for (int b = 0; b < NB; ++b)
#pragma unroll
      for (int r = 0; r < 16; ++r) o[b][r] = 0.f;
    float z = 0.f;
    while (more) {
      typename M::V v0, v1;
      load_v<T, D>(v0, Vh, s, u, 0, L);
      if (kF32 && D == 64) load_v<T, D>(v1, Vh, s, u, 1, L);
      const uint32_t bits = s.bits(u);
      float p[16];
#pragma unroll
      for (int r = 0; r < 16; ++r) p[r] = exp_from(acc0[r] * scale, mu) * inv;
      if (!u.full) {   // 0 where the row lacks the key
        const unsigned word = bits >> (4 * s.h);
#pragma unroll
        for (int r = 0; r < 16; ++r)
          p[r] = __builtin_bit_cast(
              float, __builtin_bit_cast(int, p[r]) &
                         __builtin_amdgcn_sbfe((int)word, 8 * (r >> 2) + (r & 3), 1));
      }
      Unit nnu;
      bool nnext = false;
      if (next) {
        wait_loads();
        load_k<T, D>(k, kst, s);
        acc0 = M::dot(k, q);
        nnext = it.next(nnu);
        if (nnext) fetch_k<T, D>(kst, Kh, s, nnu, L);
      }
      check_v<T, D>(z, v0, u);
      M::pv(o, v0, p, 0);
      if (!kF32 || D != 64) load_v<T, D>(v1, Vh, s, u, 1, L);
      check_v<T, D>(z, v1, u);
      M::pv(o, v1, p, 1);
      if (OUT) write_values(Ph, nnz, p, bits, u, unit_pos(rrs[s.qi], row_begin, u), s, vst);
      if (OUT == 2)
        // a register holds one key of 32 rows, neighbours in the column: its store
        // covers 128 bytes of it (of two, one per half)
        for_each_place(s.row_valid ? bits : 0u, nnz, u, cols, s, L, vst, [&](int r, int at) {
          *(float*)((char*)(Pt + (size_t)blockIdx.x * nnz) + 4u * (unsigned)at) = p[r];
        });
      u = nu, nu = nnu, more = next, next = nnext;
    }
    if constexpr (kF32) {
      // weights of 1 at most: only V can take a sum out of fp32's range
      __syncthreads();
      if (z != z) sh.redo = 1;
      __syncthreads();
      if (sh.redo) {   // from the P just written
        __threadfence_block();
        for (int r = s.wave; r < kWaveRows; r += kWavesPerGroup) {
          const int i = __builtin_amdgcn_readlane(s.row_valid ? s.row : -1, r);
          if (i >= 0)
            spmm_row<D, OutT, false>(i, s.lane, runs, row_ptr, cols, L, nnz, Ph, V + head, O + head);
        }
        __syncthreads();
        continue;
      }
    }
    combine<D, false, OutT>(
        sh, o, s, O + head, [](int, int) { return 1.f; }, [](int) {});
    __syncthreads();   // LDS is reused by the next slice
  }
}

#ifdef SPLAT_DEBUG_BOUNDS
// One index check on the device (the checked build's own test): out = the
// checked index.
__global__ void k_bounds_probe(int kind, int index, int n, int* out) {
  *out = dbg::idx(index, n, (dbg::Kind)kind);
}
#endif

// --------------------------------------------------------------- launches
// Grid: x over batch*head, so that with B*H a multiple of 8 a head's
// workgroups share one XCD's L2; y over slices, heaviest groups first.
inline int slices(const DevAcsr& a) { return a.n_groups * kWavesPerGroup; }
inline dim3 slice_grid(const DevAcsr& a, int BH) {
  const int n = slices(a);
  return dim3((unsigned)BH, (unsigned)(n < kMaxGridY ? n : kMaxGridY));
}

// Estimated times, in us beyond a launch's own 2.5 to 3.2, by which a launch
// chooses its kernel; fitted to 39 fp32 launches (4 k to 13 M non-zeros over
// all heads, every mask family, d = 64 and 128).
struct Size {
  double w, R, E, C, NS;   // d / 64; rows, non-zeros, computed scores and slices of all heads
  double longest, chain;   // the longest row's keys, the longest slice's tiles in pairs
  Size(const DevAcsr& a, int BH, int d)
      : w(d / 64.0), R((double)a.L * BH), E((double)a.nnz * BH), C((double)a.computed * BH),
        NS((double)kWavesPerGroup * a.n_groups * BH), longest(a.max_row_nnz),
        chain((a.max_slice_tiles + 1) / 2) {}
};
// At throughput a cost per slice and per computed score; else the longest slice.
double slices_us(const Size& z, double per_slice, double per_score, double chain) {
  return fmax(1e-3 * per_slice * z.NS + 1e-6 * per_score * z.w * z.C, chain);
}
// Fused, measured with a wavefront per row against slices: window 16, L = 256,
// one head 4.9 / 7.3; strided+local 8 / 64, L = 512, one head 4.5 / 10.0;
// window 16, L = 1024, 4 heads 9.1 / 7.4; blocked 64, L = 512, 4 heads 15.1 / 7.2.
bool fused_rows_faster(const Size& z) {
  return fmax(0.65e-3 * z.R + 0.035e-3 * z.w * z.E, 0.052 * z.w * z.longest) <
         slices_us(z, 16, 2.5, z.w * (1.6 + 2.6 * z.chain));
}
// R-SDDMM, where a wavefront per row pays only while the launch is bound by
// latency: window 16, L = 256, one head 2.6 / 6.1, L = 4096 6.9 / 6.3;
// strided+local 8 / 64, L = 2048, one head 4.9 / 8.6, 12 heads 36 / 17.
double rsddmm_rows_us(const Size& z) {
  return fmax(0.5e-3 * z.R + 0.027e-3 * z.w * z.E, 0.9 * z.w * ceil(z.longest / 64));
}
double rsddmm_slices_us(const Size& z) {
  return slices_us(z, 5.5, 2.2, (z.w + 1) / 2 * (2.2 + 2.4 * z.chain));
}
bool rsddmm_rows_faster(const Size& z) {
  return z.R <= 4096 && rsddmm_rows_us(z) < rsddmm_slices_us(z);
}
// R-SpMM, where a wavefront per row reads V and P in whole lines and pays over
// a wider range: window 16, L = 256, one head 3.0 / 6.1; strided+local 8 / 64,
// L = 2048, 12 heads 14 / 16.5; strided+local 128, L = 2048, 12 heads 36.5 /
// 20.6; full, L = 128, d = 128, 4 heads 5.6 / 7.2.
double rspmm_rows_us(const Size& z) {
  return fmax(0.25e-3 * z.R + 0.0085e-3 * z.w * z.E, 0.022 * z.w * z.longest);
}
double rspmm_slices_us(const Size& z) {
  return slices_us(z, 7.5, 2.2, (z.w + 1) / 2 * (2.2 + 2.4 * z.chain));
}
bool rspmm_rows_faster(const Size& z) { return rspmm_rows_us(z) < rspmm_slices_us(z); }

// bf16 steps: slices against the 128-row kernels over tiles, which share each K
// or V tile between four wavefronts and write S in whole 128-byte lines, but
// walk a group's tiles one after the other.  Measured, tiles against slices:
// R-SDDMM window 512 + 64 global, L = 4096, 16 heads 178 / 91 us, 64 heads 286 /
// 349; blocked 64, L = 1024, 16 heads 9.4 / 5.9; window 4, d = 128, L = 1024, 16
// heads 14.7 / 6.9, 64 heads 18.6 / 20.7.  Past the caches (192 MB; twice that
// where rows begin and end on lines) the slices' partial lines cost: window 128,
// L = 4096, 64 heads 102 / 130, full, L = 1024, 64 heads 98 / 70, L = 2048, 32
// heads 145 / 168.  Rows that begin and end on lines suit the tile kernel best
// where its walk is short and the chip is full: full, L = 384, 402 heads 58 / 75,
// L = 448, 382 heads 69 / 100, window 540, L = 352, 211 heads 29 / 36 (against: full, L =
// 352, 304 heads 49 / 37; of 28 such launches 22 are faster over tiles by more than
// 5%, 6 slower).
bool rsddmm_bf16_slices(const DevAcsr& a, const Size& z) {
  const double k = (z.w + 1) / 2;
  if (a.rows_aligned && a.max_group_tiles <= 11 && z.NS >= 1800) return false;
  const double value = z.E > (a.rows_aligned ? 96e6 : 48e6) ? 1.4e-6 : 0.75e-6;
  const double slc =
      2.5 + k * fmax(0.7 + 1.45 * z.chain, 5e-3 * z.NS + value * z.E);
  const double tiles =
      2.5 + fmax(3 + 2.75 * a.max_group_tiles, 3.5e-3 * z.NS + 1e-6 * k * z.E);
  return slc < tiles;
}
// R-SpMM window 512 + 64 global, L = 4096, 16 heads 130 / 80 us, 64 heads 267 /
// 318; blocked 64, L = 1024, 16 heads 7.7 / 5.9; full, L = 1024, 64 heads 48 / 71;
// L = 218, 113 heads 10.4 / 14.4; groups of one tile: dilated 13 / 6, L = 151, 25
// heads 4.2 / 5.4, d = 128, dilated 24 / 6, L = 116, 30 heads 4.6 / 5.8.  One
// choice for both layouts, whose results are the same bits.  Column-major values
// cost the tile kernel more (dilated 40 / 3, L = 4106, 3 heads, d = 128 27 / 13), so
// a handle that has them takes the slices further, but at d = 64 not for groups of
// one tile (5.1 / 5.7), nor for columns that step beyond a chip's slices (dilated
// 51 / 4, L = 947, 28 heads 14.1 / 19.1), whose places are looked up one by one.
bool rspmm_bf16_slices(const DevAcsr& a, const Size& z) {
  const double k = (z.w + 1) / 2;
  if (a.max_group_tiles <= 1 && !(a.columns && z.w == 2)) return false;
  if (a.columns_step && z.w == 1 && z.NS > 768) return false;
  const double group =
      a.columns ? 4.5 + 2 * a.max_group_tiles : 2 + z.w / 2 + 2.2 * a.max_group_tiles;
  const double slc =
      2.5 + fmax(0.9 + 1.5 * k * z.chain, k * (4.5e-3 * z.NS + 1.1e-6 * z.C));
  const double tiles = 2 + fmax(group, 3.5e-3 * z.NS + 0.75e-6 * k * z.C);
  return slc < tiles;
}

// bf16, one kernel against the steps: blocked 64, L = 1024, 16 heads 9.9 /
// 26.5 us, window 512 + 64 global, L = 4096, 64 heads 569 / 1006.  The kernel
// forms the scores twice and costs more a slice; the steps cost two launches
// more, and stores and reads of S.  Many slices of few non-zeros pay for the
// steps: d = 64, window 4, L = 12000, 57 heads 256 / 209, window 8, 19040 slices
// 230 / 207, window 13, 24420 slices 285 / 264; d = 128, window 8, L = 8192, 32
// heads 161 / 137, blocked 6, 8064 slices 149 / 116, window 31, L = 6830, 51 heads
// 240 / 228; below 5000 and 2500 slices the launches decide (d = 128, blocked 6,
// 2324 slices 49 / 53).  The lines are fitted to 1160 launches, of which 9 lose
// more than 5% by them (14% at most).  A long row group holds the steps up.  The
// column-major branch has a fourth launch (window 15, dilation 3, L = 2900, 136
// heads 236 / 254), and O alone costs less than O and P (values: P is stored;
// d = 64, window 4, L = 12000, 57 heads 197 / 209; d = 128, dilated 8 / 5, L =
// 16288, 37 heads 322 / 306): there only the thinnest masks.  fp32: strided+local
// 128, L = 2048, 12 heads 39.5 / 50.6; window 16, L = 256, one head 9.8 / 8.5; at d
// = 128, where one workgroup's LDS fills a CU, window 1, L = 925, 19 heads 41 / 29,
// full, L = 1523, 18 heads 426 / 336, dilated 12 / 5, L = 1968, 42 heads 144 / 117,
// but a long group holds the steps up more (window 11 + 2 global, L = 1638, 48 heads
// 194 / 257), and the column-major branch has its fourth launch (full, L = 968, 7
// heads 84 / 123).
bool chain_faster(const DevAcsr& a, int dtype, int BH, int d, bool col, bool values) {
  const Size z(a, BH, d);
  if (dtype != 0) {
    if (z.C > 16 * z.E && z.NS > 4096) return false;
    const double few = values ? (d == 64 ? 1200 * (z.NS - 5000) : 2700 * (z.NS - 2500))
                              : (d == 64 ? 0 : 1400 * (z.NS - 5000));
    return col || z.E >= few || a.max_group_tiles > 16;
  }
  const double steps =
      7.8 + 1.6e-6 * z.E +
      (rsddmm_rows_faster(z) ? rsddmm_rows_us(z) : rsddmm_slices_us(z)) +
      fmin(rspmm_rows_us(z), rspmm_slices_us(z));
  const double walk = (z.w + 1) / 2 * (1.2 + 5.6 * z.chain);
  const int64_t longest = (int64_t)a.max_group_tiles * a.n_groups;
  const bool alone = d == 128 && !col && longest <= 2 * (int64_t)a.n_tiles;
  return 3.2 + (alone ? slices_us(z, 15, 5.5, walk) : slices_us(z, 10, 4.2, walk)) < steps;
}

}  // namespace

Route rsddmm_route(const DevAcsr& a, int dtype, int BH, int d) {
  const Size z(a, BH, d);
  if (dtype != 0) return rsddmm_bf16_slices(a, z) ? kRouteSlices : kRouteTiles;
  return rsddmm_rows_faster(z) ? kRouteRows : kRouteSlices;
}
Route rspmm_route(const DevAcsr& a, int dtype, int BH, int d) {
  const Size z(a, BH, d);
  if (dtype != 0) return rspmm_bf16_slices(a, z) ? kRouteSlices : kRouteTiles;
  return rspmm_rows_faster(z) ? kRouteRows : kRouteSlices;
}
Route fused_f32_route(const DevAcsr& a, int BH, int d) {
  return fused_rows_faster(Size(a, BH, d)) ? kRouteRows : kRouteSlices;
}
Route unfused_route(const DevAcsr& a, int dtype, int BH, int d, bool col, bool values) {
  return chain_faster(a, dtype, BH, d, col, values) ? kRouteChain : kRouteSteps;
}

namespace {

// Grid of the row kernels: four rows per workgroup.
inline dim3 row_grid(const DevAcsr& a, int BH) {
  return dim3((unsigned)BH, (unsigned)((a.L + 3) / 4));
}

template <int D, typename OutT>
hipError_t fused_rows(const DevAcsr& a, int BH, const void* Q, const void* K, const void* V,
                      float scale, void* O, hipStream_t st) {
  hipLaunchKernelGGL((k_fused_rows<D, OutT>), row_grid(a, BH), dim3(kThreads), 0, st,
                     a.row_ptr, a.runs, a.L, (const float*)Q,
                     (const float*)K, (const float*)V, scale, (OutT*)O);
  return hipGetLastError();
}

template <int D>
hipError_t fused_d(const DevAcsr& a, int BH, const void* Q, const void* K, const void* V,
                   float scale, void* O, int out_dtype, hipStream_t st) {
  if (fused_f32_route(a, BH, D) == kRouteRows)
    return out_dtype == 0 ? fused_rows<D, float>(a, BH, Q, K, V, scale, O, st)
                          : fused_rows<D, __bf16>(a, BH, Q, K, V, scale, O, st);
  if (out_dtype == 0)
    hipLaunchKernelGGL((k_fused_slices<D, float>), slice_grid(a, BH), dim3(kThreads), 0, st,
                       a.groups, a.rows, a.row_ptr, a.runs, a.tiles, a.masks, a.L, slices(a),
                       (const float*)Q, (const float*)K, (const float*)V, scale, (float*)O);
  else
    hipLaunchKernelGGL((k_fused_slices<D, __bf16>), slice_grid(a, BH), dim3(kThreads), 0, st,
                       a.groups, a.rows, a.row_ptr, a.runs, a.tiles, a.masks, a.L, slices(a),
                       (const float*)Q, (const float*)K, (const float*)V, scale, (__bf16*)O);
  return hipGetLastError();
}

template <typename T, int D>
hipError_t rsddmm_d(const DevAcsr& a, int BH, const void* Q, const void* K, float scale, float* S,
                    hipStream_t st) {
  if constexpr (sizeof(T) == 4)
    if (rsddmm_route(a, 0, BH, D) == kRouteRows) {
      hipLaunchKernelGGL((k_rsddmm_rows<D>), dim3(a.L, BH), dim3(64), 0, st, a.row_ptr, a.runs, a.L,
                         a.nnz, (const float*)Q, (const float*)K, scale, S);
      return hipGetLastError();
    }
  hipLaunchKernelGGL((k_rsddmm_slices<T, D>), slice_grid(a, BH), dim3(kThreads), 0, st, a.groups,
                     a.rows, a.row_ptr, a.runs, a.tiles, a.masks, a.L, a.nnz, slices(a),
                     (const T*)Q, (const T*)K, scale, S);
  return hipGetLastError();
}

template <typename T, int D, typename OutT, bool COL>
hipError_t rspmm_d(const DevAcsr& a, int BH, const float* P, const void* V, void* O,
                   hipStream_t st) {
  if constexpr (sizeof(T) == 4)
    if (rspmm_route(a, 0, BH, D) == kRouteRows) {
      hipLaunchKernelGGL((k_rspmm_rows<D, OutT, COL>), dim3(a.L, BH), dim3(64), 0, st, a.row_ptr,
                         a.runs, a.cols, a.L, a.nnz, P, (const float*)V, (OutT*)O);
      return hipGetLastError();
    }
  hipLaunchKernelGGL((k_rspmm_slices<T, D, OutT, COL>), slice_grid(a, BH), dim3(kThreads), 0, st,
                     a.groups, a.rows, a.row_ptr, a.runs, a.tiles, a.masks, a.cols, a.L, a.nnz,
                     slices(a), P, (const T*)V, (OutT*)O);
  return hipGetLastError();
}

template <typename T, bool COL>
hipError_t rspmm_t(const DevAcsr& a, int BH, int d, const float* P, const void* V, void* O,
                   int out_dtype, hipStream_t st) {
  if (d == 64)
    return out_dtype == 0 ? rspmm_d<T, 64, float, COL>(a, BH, P, V, O, st)
                          : rspmm_d<T, 64, __bf16, COL>(a, BH, P, V, O, st);
  return out_dtype == 0 ? rspmm_d<T, 128, float, COL>(a, BH, P, V, O, st)
                        : rspmm_d<T, 128, __bf16, COL>(a, BH, P, V, O, st);
}

template <typename T, int D, typename OutT>
hipError_t chain_d(const DevAcsr& a, int BH, const void* Q, const void* K, const void* V,
                   float scale, float* P, float* Pt, void* O, hipStream_t st) {
  auto go = [&](auto kernel) {
    hipLaunchKernelGGL(kernel, slice_grid(a, BH), dim3(kThreads), 0, st, a.groups, a.rows,
                       a.row_ptr, a.runs, a.tiles, a.masks, a.cols, a.L, a.nnz, slices(a),
                       (const T*)Q, (const T*)K, (const T*)V, scale, P, Pt, (OutT*)O);
    return hipGetLastError();
  };
  if (Pt) return go(k_chain_slices<T, D, OutT, 2>);
  if constexpr (std::is_same<T, __bf16>::value)
    if (!P) return go(k_chain_slices<T, D, OutT, 0>);
  return go(k_chain_slices<T, D, OutT, 1>);
}

template <typename T>
hipError_t chain_t(const DevAcsr& a, int BH, int d, const void* Q, const void* K, const void* V,
                   float scale, float* P, float* Pt, void* O, int out_dtype, hipStream_t st) {
  if (d == 64)
    return out_dtype == 0 ? chain_d<T, 64, float>(a, BH, Q, K, V, scale, P, Pt, O, st)
                          : chain_d<T, 64, __bf16>(a, BH, Q, K, V, scale, P, Pt, O, st);
  return out_dtype == 0 ? chain_d<T, 128, float>(a, BH, Q, K, V, scale, P, Pt, O, st)
                        : chain_d<T, 128, __bf16>(a, BH, Q, K, V, scale, P, Pt, O, st);
}

}  // namespace

hipError_t bounds_collect_slices(uint32_t* bits, bool clear) { return dbg::collect(bits, clear); }

hipError_t bounds_probe(int kind, int index, int n, int* result) {
#ifndef SPLAT_DEBUG_BOUNDS
  (void)kind;
  (void)index;
  (void)n;
  (void)result;
  return hipErrorNotSupported;
#else
  int* d = nullptr;
  hipError_t e = hipMalloc(&d, sizeof(int));
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(k_bounds_probe, dim3(1), dim3(1), 0, 0, kind, index, n, d);
  e = hipGetLastError();
  if (e == hipSuccess) e = hipMemcpy(result, d, sizeof(int), hipMemcpyDeviceToHost);
  const hipError_t f = hipFree(d);
  return e != hipSuccess ? e : f;
#endif
}

hipError_t launch_fused_f32(const DevAcsr& a, int BH, int d, const void* Q, const void* K,
                            const void* V, float scale, void* O, int out_dtype, hipStream_t st) {
  return d == 64 ? fused_d<64>(a, BH, Q, K, V, scale, O, out_dtype, st)
                 : fused_d<128>(a, BH, Q, K, V, scale, O, out_dtype, st);
}

hipError_t launch_rsddmm(const DevAcsr& a, int dtype, int BH, int d, const void* Q, const void* K,
                         float scale, float* S, hipStream_t st) {
  if (dtype != 0) {
    if (rsddmm_route(a, dtype, BH, d) == kRouteTiles)
      return launch_rsddmm_tiles(a, BH, d, Q, K, scale, S, st);
    return d == 64 ? rsddmm_d<__bf16, 64>(a, BH, Q, K, scale, S, st)
                   : rsddmm_d<__bf16, 128>(a, BH, Q, K, scale, S, st);
  }
  return d == 64 ? rsddmm_d<float, 64>(a, BH, Q, K, scale, S, st)
                 : rsddmm_d<float, 128>(a, BH, Q, K, scale, S, st);
}

hipError_t launch_rspmm(const DevAcsr& a, int dtype, int BH, int d, const float* P, const void* V,
                        void* O, int out_dtype, bool colmajor, hipStream_t st) {
  if (dtype != 0) {
    if (rspmm_route(a, dtype, BH, d) == kRouteTiles)
      return launch_rspmm_tiles(a, BH, d, P, V, O, out_dtype, colmajor, st);
    return colmajor ? rspmm_t<__bf16, true>(a, BH, d, P, V, O, out_dtype, st)
                    : rspmm_t<__bf16, false>(a, BH, d, P, V, O, out_dtype, st);
  }
  return colmajor ? rspmm_t<float, true>(a, BH, d, P, V, O, out_dtype, st)
                  : rspmm_t<float, false>(a, BH, d, P, V, O, out_dtype, st);
}

hipError_t launch_chain(const DevAcsr& a, int dtype, int BH, int d, const void* Q, const void* K,
                        const void* V, float scale, float* P, float* Pt, void* O, int out_dtype,
                        hipStream_t st) {
  return dtype == 0 ? chain_t<float>(a, BH, d, Q, K, V, scale, P, Pt, O, out_dtype, st)
                    : chain_t<__bf16>(a, BH, d, Q, K, V, scale, P, Pt, O, out_dtype, st);
}

}  // namespace splat
