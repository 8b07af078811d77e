// softmax_prefix.hip -- exact softmax attention of the active block over a
// request's cached prefix plus the block itself: the softmax layer that the
// hybrid layer replaces (Section 2.2 attention without a mask inside the
// block; the comparison of the paper's kernel benchmark, Appendix A).
//
// Split-KV flash decoding.  Keys are indexed in the concatenation
// [k_cache[b][0 .. P_b-1]; k_block[b][0 .. L-1]] and cut into ranges of whole
// 32-key tiles, as many per request as its length asks for (SpPlan).
// One workgroup per (request b, KV head g, range s) with one wave per query
// head of the group (GQA packing: the G heads share every K/V tile through
// LDS).  Each 32-key tile gives Sc^T = K Q^T (keys in rows, one query per
// lane column), an online-softmax update, and O^T += V^T P^T, with P rounded
// once to the operand type and the running sum taken over the rounded
// weights.  A second kernel merges the ranges with their log-sum-exp weights;
// with a single range the first kernel writes the normalised output itself.
//
// The cache is either contiguous per request ([B][max_prefix][Hkv][d]) or
// paged: a pool of fixed-size pages ([n_pages][page][Hkv][d]) and a page table
// per request, as a serving engine's paged KV cache keeps it (Section 3.3).
// The page size is a power of two of at least 32 rows, so a 32-key tile lies
// in one page.  The ring kernel stages its range's page numbers in LDS when
// it starts (a range holds at most kMaxRange keys), so the copies of a tile
// take their page from LDS and no vector load of the page table sits among
// the copies whose counts the ring waits on.
#include <algorithm>
#include <type_traits>

#include "device.h"
#include "launch.h"

namespace hyb {

template <typename T, int D, int NG>
struct SpCfg {
  typedef Mma<T> M;
  typedef typename M::op_t op_t;
  static constexpr int KD = D / M::KW;
  static constexpr int KL = kTile / M::KW;
  static constexpr int NCT = D / kTile;
  static constexpr int EPC = 16 / (int)sizeof(T);  // elements per 16 bytes
  static constexpr int KLD = D + EPC;              // K rows: 16-byte pad
  static constexpr int VLD = D + 2 * EPC;          // V rows: 32-byte pad
  static constexpr int CPR = D / EPC;              // 16-byte chunks per row
  static constexpr int NCH = (kTile * CPR + kWave * NG - 1) / (kWave * NG);  // per thread
  struct alignas(16) Smem {
    T k[2][kTile][KLD];
    T v[2][kTile][VLD];
  };
};

constexpr int kMaxGroup = 8;  // query heads per KV head handled by one WG
// Keys of one split range at most: 32768 cached keys and a block fit one, and
// the page numbers of so many leave room for four of the paged ring's
// workgroups on a CU at d = 64 (65536 would leave room for three).
constexpr int kMaxRange = 49152;
// pages of one range at the smallest page size (32), unaligned ends included
constexpr int kMaxRangePages = kMaxRange / 32 + 2;

// Page of cached token j of a request (page table row ptab), clamped to the
// pool.
__device__ inline int sp_page(const SoftmaxPrefixArgs& a, const int32_t* ptab, int j) {
  const int pg = ptab[j >> a.page_shift];
  return min(max(pg, 0), a.n_pages - 1);
}

// Keys of request b: its cached prefix (clamped) and the block.
__device__ inline int sp_keys(const SoftmaxPrefixArgs& a, int b) {
  return min(max(a.prefix_len[b], 0), a.max_prefix) + a.s.L;
}

__device__ inline int sp_tiles(const SoftmaxPrefixArgs& a, int b) {
  return (sp_keys(a, b) + kTile - 1) / kTile;
}

// How the requests' keys are cut.  The lengths are known on the device only,
// so every workgroup works the cut out for itself, from prefix_len alone and
// with the same result: request b gets ceil(tiles_b / c) ranges, numbered
// through over the requests (so that the workgroups that have a range come first
// and spread over the chip; a fixed number of places per request took 8 paged
// requests of 1 to 4096 keys from 29 to 34 us), and range s of request b takes
// an even share of its tiles.  The tiles per range c is the
// candidate with the least estimated time (in whole numbers, so that every kernel
// finds the same).  Per KV head, `sat` workgroups use the memory fully and the
// chip holds `slots` of them at once.  Up to `sat` ranges take the time of the
// longest.  More, as far as they all fit, share the memory: the time of all their
// tiles (a tenth more, as they don't end together), or of the longest among as
// many neighbours as its CU has, half of whom end early, if that is more.  Ranges
// beyond that also pay for the part of the last round that stays empty.  A range
// costs its start, its partial result and that result's merge besides its tiles
// (sp_range_cost).  Candidates lie around the even share of `sat`; the
// last one cuts the longest request into limit / B ranges, so that all ranges fit
// the grid and the workspace.
// Equal cuts of max_prefix into n_split ranges, as it was, make 2048
// workgroups whatever the lengths: four rounds and a merge where one round of
// whole requests fills the chip (128 requests of 32768 keys: 1.70 against
// 1.54 ms, the loop below included), and ranges past a short request's end
// that still write, and have merged, an empty result (24 requests of 1 to
// 8192 keys: 104 against 76 us; 8 of 32768: 232 against 137 us).
struct SpCut {
  int slots, sat, limit;
  int layer;  // ranges per KV head that give every CU one workgroup
  int c;      // tiles per range where the host cuts, else 0
};
struct SpPlan {
  int c;       // tiles per range, before the even share
  bool whole;  // every request is one range
};
constexpr int kCand = 16;        // candidates; kWave / kCand = 4 lanes share one
constexpr int kPlanTiles = 256;  // requests staged in LDS at most

// A range's cost in tiles: its start (a tile of d = 64 is half as long) and the
// fp32 rows of its G heads and L queries, written and read once; at most ten.
__device__ inline int sp_range_cost(const SoftmaxPrefixArgs& a) {
  return min(10, (a.s.D == 128 ? 2 : 4) + a.s.Hq / a.s.Hkv * a.s.L / (a.s.dtype == 1 ? 16 : 32));
}

// Sum or maximum over the wave, in every lane: rotations within the rows of 16
// lanes, then exchanges of rows.  (Six shuffles through LDS took 0.3 us, and a
// plan and its use are several of these.)
template <typename Op>
__device__ inline int wave_all(int x, Op op) {
  x = op(x, __builtin_amdgcn_update_dpp(0, x, 0x128, 0xf, 0xf, false));  // row_ror:8
  x = op(x, __builtin_amdgcn_update_dpp(0, x, 0x124, 0xf, 0xf, false));
  x = op(x, __builtin_amdgcn_update_dpp(0, x, 0x122, 0xf, 0xf, false));
  x = op(x, __builtin_amdgcn_update_dpp(0, x, 0x121, 0xf, 0xf, false));
  auto f = [](int v) { return __builtin_bit_cast(float, v); };
  x = op(x, __builtin_bit_cast(int, xor16(f(x))));
  return op(x, __builtin_bit_cast(int, xor32(f(x))));
}
struct AddOp {
  __device__ int operator()(int a, int b) const { return a + b; }
};
struct MaxOp {
  __device__ int operator()(int a, int b) const { return max(a, b); }
};
struct MinOp {
  __device__ int operator()(int a, int b) const { return min(a, b); }
};
// Sum over the lanes up to this one.
__device__ inline int wave_scan(int x) {
  x += __builtin_amdgcn_update_dpp(0, x, 0x111, 0xf, 0xf, true);  // row_shr:1
  x += __builtin_amdgcn_update_dpp(0, x, 0x112, 0xf, 0xf, true);
  x += __builtin_amdgcn_update_dpp(0, x, 0x114, 0xf, 0xf, true);
  x += __builtin_amdgcn_update_dpp(0, x, 0x118, 0xf, 0xf, true);
  x += __builtin_amdgcn_update_dpp(0, x, 0x142, 0xa, 0xf, false);  // row_bcast:15 into rows 1, 3
  x += __builtin_amdgcn_update_dpp(0, x, 0x143, 0xc, 0xf, false);  // row_bcast:31 into rows 2, 3
  return x;
}

// tiles: LDS scratch of kPlanInts ints.  All threads of the workgroup; the
// first wave plans.  (The scratch is part of a tile buffer that is first written
// behind a later barrier: on its own it would cost d = 64 one of five workgroups
// on a CU.)
constexpr int kPlanInts = kPlanTiles + 2;
__device__ inline SpPlan sp_plan(const SoftmaxPrefixArgs& a, const SpCut& cut, int* tiles) {
  const int B = a.s.B, tid = threadIdx.x;
  if (a.n_split == 1) return SpPlan{1 << 24, true};
  if (cut.c > 0) return SpPlan{cut.c, false};
  if (tid < kWave) {
    int total = 0, most = 0;
    const int end = B <= kPlanTiles ? (B + 15) & ~15 : B;  // (padded with empty requests)
    for (int b0 = tid; b0 < end; b0 += kWave) {
      const int nt = b0 < B ? sp_tiles(a, b0) : 0;
      if (B <= kPlanTiles) tiles[b0] = nt;
      total += nt;
      most = max(most, nt);
    }
    total = __builtin_amdgcn_readfirstlane(wave_all(total, AddOp{}));
    most = __builtin_amdgcn_readfirstlane(wave_all(most, MaxOp{}));
    // (tiles: written and read by this wave)
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront", "local");
    const int share = max(1, (total + cut.sat - 1) / cut.sat);
    const int cand = tid % kCand, sub = tid / kCand;
    // 1/4, 1/3, 1/2, 3/4, then from 1 on in steps of 1/16 to 1 1/2, 2, 4
    const int num = cand < 4 ? (cand == 0 ? 12 : cand == 1 ? 16 : cand == 2 ? 24 : 36)
                    : cand < 13 ? 48 + 3 * (cand - 4) : cand == 13 ? 96 : 192;
    int c = (int)(((long)share * num + 47) / 48);
    c = min(max(c, 4), kMaxRange / kTile);
    const int least = max(1, cut.limit / B);
    if (cand == kCand - 1) c = (most + least - 1) / least;
    // the candidate's ranges: x / c by a reciprocal, within one of it, so that
    // the correction leaves one too many at worst and never too few (c times the
    // quotient's error is below one for x up to 5 million); exact beyond
    const float rc = 1.0f / (float)c;
    auto ranges = [&](int x) {
      if (x >= 1 << 20) return (x + c - 1) / c;
      const int n = (int)((float)x * rc);
      return n + (n * c < x ? 1 : 0);
    };
    int sum = 0;
    if (B <= kPlanTiles) {
      for (int b0 = 4 * sub; b0 < end; b0 += 16) {
        const int4 x = *reinterpret_cast<const int4*>(tiles + b0);
        sum += ranges(x.x) + ranges(x.y) + ranges(x.z) + ranges(x.w);
      }
    } else {
      for (int b0 = sub; b0 < B; b0 += kWave / kCand) sum += ranges(sp_tiles(a, b0));
    }
    static_assert(kCand == 16, "the lanes that share a candidate are a row apart");
    sum += __builtin_bit_cast(int, xor16(__builtin_bit_cast(float, sum)));
    sum += __builtin_bit_cast(int, xor32(__builtin_bit_cast(float, sum)));
    const int extra = sum > B ? sp_range_cost(a) : 0, longest = min(c, most) + extra;
    const int work = (min(total, 1 << 26) + sum * extra) * 11 / 10, rest = sum % cut.slots;
    int time = longest * cut.sat;
    if (sum > cut.slots)
      time = work + (rest > 0 ? time * (cut.slots - rest) / cut.slots : 0);
    else if (sum > cut.sat)
      time = max(longest * (cut.sat + (sum + cut.layer - 1) / cut.layer * cut.layer) / 2, work);
    const int cost = sum <= cut.limit ? time : cand == kCand - 1 ? 0x7ffffffe : 0x7fffffff;
    const int at = __builtin_ctzll(__ballot(cost == wave_all(cost, MinOp{})));
    const int pick = __builtin_amdgcn_readlane(c, at);
    if (tid == 0) {
      tiles[kPlanTiles] = pick;
      tiles[kPlanTiles + 1] = most <= pick;
    }
  }
  __syncthreads();
  return SpPlan{__builtin_amdgcn_readfirstlane(tiles[kPlanTiles]),
                __builtin_amdgcn_readfirstlane(tiles[kPlanTiles + 1]) != 0};
}

// Ranges of a request of nt tiles.
__device__ inline int sp_ranges(const SpPlan& p, int nt) { return (nt + p.c - 1) / p.c; }

// Range number r of the plan: its request, its place there, how many ranges
// that request has and its keys lo .. hi-1.  b = -1: no such range.  Where every
// request is one range, that is request r; else the ranges of the requests
// before are summed, 64 requests at a time.  (Summed in every case, calls of
// many short requests paid for it: 4096 requests of 64 keys 907 us, now 377;
// 4096 of 32 at 8 KV heads of d = 64 584 us, now 141.)
struct SpRange {
  int b, s, n, lo, hi;
};
__device__ inline SpRange sp_share(const SoftmaxPrefixArgs& a, int b, int s, int n) {
  // an even share of the tiles: the first tiles % n ranges take one more
  const int keys = sp_keys(a, b), tiles = (keys + kTile - 1) / kTile;
  const int each = tiles / n, more = tiles % n;
  const int t0 = s * each + min(s, more);
  return SpRange{b, s, n, t0 * kTile, min((t0 + each + (s < more ? 1 : 0)) * kTile, keys)};
}
__device__ inline SpRange sp_range(const SoftmaxPrefixArgs& a, const SpPlan& p, int r, int lane) {
  const int B = a.s.B;
  const SpRange none{-1, 0, 0, 0, 0};
  if (p.whole) return r < B ? SpRange{r, 0, 1, 0, sp_keys(a, r)} : none;
  int base = 0;
  for (int b0 = 0; b0 < B; b0 += kWave) {
    const int n = b0 + lane < B ? sp_ranges(p, sp_tiles(a, b0 + lane)) : 0;
    const int end = wave_scan(n);
    const int all = __builtin_amdgcn_readlane(end, kWave - 1);
    if (r < base + all) {
      const int at = __builtin_ctzll(__ballot(r < base + end));
      const int nb = __builtin_amdgcn_readlane(n, at);
      return sp_share(a, b0 + at, r - base - (__builtin_amdgcn_readlane(end, at) - nb), nb);
    }
    base += all;
  }
  return none;
}

// Partial results in the workspace, by range number r: rows of D floats
// [r][head][query], then (max, sum) pairs in the same order; at most n_split
// ranges per request on average.
__device__ inline size_t sp_row(const SoftmaxPrefixArgs& a, int r, int h, int i) {
  return ((size_t)r * a.s.Hq + h) * a.s.L + i;
}
template <int D>
__device__ inline float* sp_ml(const SoftmaxPrefixArgs& a) {
  return (float*)a.ws + (size_t)a.s.B * a.n_split * a.s.Hq * a.s.L * D;
}

// The reference of a query's weights 2^(s - ref), in the log2 domain.  P enters
// P V rounded to bf16, and a weight that is a power of two does not round; so
// the heaviest weights, those that make a row, round least if the references
// have the fractions of the maxima of many tiles.  With one running maximum per
// range the error therefore grows with the range's length (rms of the weights'
// part over 512, 8224 and 32800 normal keys: 1.42, 1.59 and 1.63e-3).  So a tile
// may restart the reference at its own maximum, moved up by whole powers of two
// to at least the maximum so far (no accumulator grows), and in between a
// larger maximum raises it.  A restart costs a rescale of the accumulators.
// Where a maximum is young, tiles rescale anyway (some of a wave's 32 queries
// rises in two of three tiles up to the 32nd): there every tile restarts, later
// every fourth (1.17 and 1.54e-3: less than any range of a quarter or an eighth of
// the length, which is how much shorter equal cuts of the longest prefix are).
// The register-staged kernel, which waits for its own arithmetic, restarts at
// every second of the early tiles (1.41e-3).
// Error against 64 bits, bf16 outputs included, and time of 128 x 32768 keys:
// 2.25e-3 and 1531 us, with one running maximum per range 2.32e-3 and 1528 us,
// with a restart at every tile throughout 2.1e-3 and 1710 us; 24 paged requests
// of 1 to 8192: 2.0e-3 and 70 us, and 2.2e-3 and 71 us.
struct SpRef {
  float most = -INFINITY;  // maximum so far
  float ref = -INFINITY;
  template <int kEarly>
  __device__ static inline bool restarts(int n) { return n < 64 ? n % kEarly == 0 : n % 4 == 0; }
  // Takes a tile's maximum; true where some lane's reference moves, to next
  // (what it was is left in ref for the rescale, and set by the caller).
  __device__ inline bool take(float mt, bool restart, float& next) {
    most = fmaxf(most, mt);
    if (restart) {  // uniform
      const float w = fmaxf(mt, most - 100.0f);  // (finite after a finite tile)
      next = w + fmaxf(0.0f, ceilf(most - w));
    } else {
      next = fmaxf(ref, mt);
    }
    return __any(next != ref);
  }
};

// One wave per query head of the KV group; 32-key tiles double-buffered in
// LDS: the tile after next is loaded into registers while the current one is
// computed, and the next one is moved from registers into the free buffer at
// the end of the step, so one barrier per tile orders everything.
template <typename T, int D, int NG, bool PAGED>
__global__ __launch_bounds__(kWave* NG) void hyb_sp_partial_kernel(
    SoftmaxPrefixArgs a, SpCut cut) {
  typedef SpCfg<T, D, NG> C;
  typedef typename C::M M;
  typedef typename C::op_t op_t;
  constexpr int E = M::E, KW = M::KW, EPC = C::EPC, CPR = C::CPR, NCH = C::NCH;
  __shared__ typename C::Smem sh;

  const int tid = threadIdx.x, lane = tid & (kWave - 1);
  const int w = __builtin_amdgcn_readfirstlane(tid / kWave);
  const int li = lane & 31, hh = lane >> 5;
  const int Hq = a.s.Hq, Hkv = a.s.Hkv, L = a.s.L, G = Hq / Hkv;
  const int Pmax = a.max_prefix;
  const int g = blockIdx.x % Hkv, r = blockIdx.x / Hkv, h = g * G + w;
  static_assert(sizeof(sh.v[1]) >= kPlanInts * sizeof(int), "the plan's scratch fits a tile");
  const SpRange rg = sp_range(a, sp_plan(a, cut, reinterpret_cast<int*>(sh.v[1])), r, lane);
  if (rg.b < 0) return;  // uniform: past the plan's last range
  const int b = rg.b, lo = rg.lo, hi = rg.hi;
  const int P = sp_keys(a, b) - L;
  const size_t qstride = (size_t)Hq * D, kstride = (size_t)Hkv * D;

  op_t qop[C::KD];
  {
    const T* qrow = (const T*)a.q + ((size_t)b * L * Hq + h) * D +
                    (size_t)li * qstride + hh * E;
#pragma unroll
    for (int ks = 0; ks < C::KD; ++ks)
      qop[ks] = li < L ? load_op<T>(qrow + ks * KW) : M::zero();
  }
  // contiguous: this request's rows; paged: the pool, at KV head g
  const T* kc = (const T*)a.k_cache + ((PAGED ? 0 : (size_t)b * Pmax * Hkv) + g) * D;
  const T* vc = (const T*)a.v_cache + ((PAGED ? 0 : (size_t)b * Pmax * Hkv) + g) * D;
  const T* kbk = (const T*)a.k + ((size_t)b * L * Hkv + g) * D;
  const T* vbk = (const T*)a.v + ((size_t)b * L * Hkv + g) * D;
  const int32_t* ptab = PAGED ? a.page_table + (size_t)b * a.max_pages : nullptr;
  // row offset of cached token j (j < P)
  auto crow = [&](int j) __attribute__((always_inline)) -> size_t {
    if constexpr (PAGED)
      return (((size_t)sp_page(a, ptab, j) << a.page_shift) + (j & ((1 << a.page_shift) - 1))) *
             kstride;
    else
      return (size_t)j * kstride;
  };

  // Tile loads: keys past the range read the range's last key (in bounds)
  // and are masked out of the scores below.
  // A tile's share of this thread, held in registers between its load and
  // its move into LDS: nx is the next tile, af the one after it.
  struct TileRegs {
    uint4 k[NCH], v[NCH];
  };
  auto fetch = [&](int j0) __attribute__((always_inline)) {
    TileRegs r;
#pragma unroll
    for (int c = 0; c < NCH; ++c) {
      const int idx = tid + c * kWave * NG, key = idx / CPR, part = idx % CPR;
      if (idx < kTile * CPR) {  // (NG not a power of two: a partial last set)
        const int j = min(j0 + key, hi - 1);
        const size_t o = (size_t)part * EPC;
        const size_t cr = j < P ? crow(j) : 0;
        const T* ks = j < P ? kc + cr : kbk + (size_t)(j - P) * kstride;
        const T* vs = j < P ? vc + cr : vbk + (size_t)(j - P) * kstride;
        r.k[c] = *reinterpret_cast<const uint4*>(ks + o);
        r.v[c] = *reinterpret_cast<const uint4*>(vs + o);
      }
    }
    return r;
  };
  auto put = [&](const TileRegs& r, int buf) __attribute__((always_inline)) {
#pragma unroll
    for (int c = 0; c < NCH; ++c) {
      const int idx = tid + c * kWave * NG, key = idx / CPR, part = idx % CPR;
      if (idx < kTile * CPR) {
        *reinterpret_cast<uint4*>(&sh.k[buf][key][part * EPC]) = r.k[c];
        *reinterpret_cast<uint4*>(&sh.v[buf][key][part * EPC]) = r.v[c];
      }
    }
  };
  // V^T operand of column tile ct, k-step ks: lane (li, hh) holds column
  // ct*32 + li at keys row_of(ks*E + e, hh).  bf16: in each 16-lane quarter
  // the transposing read gives lane i element i%4 of the 8-byte pieces
  // addressed by lanes i/4 + 4j (j = 0..3); lane i addresses key
  // kb + i/4 at columns cb + 4*(i%4) .. +3, so it receives keys kb .. kb+3
  // of column cb + i.
  auto vt_op = [&](int buf, int ct, int ks) __attribute__((always_inline)) -> op_t {
    if constexpr (E == 1) {
      return to_f32(sh.v[buf][row_of(ks, hh)][ct * kTile + li]);
    } else {
      typedef short s16x4 __attribute__((ext_vector_type(4)));
      const int i = lane & 15;
      const int cb = ct * kTile + 16 * ((lane >> 4) & 1);
      const int kb = 16 * ks + 4 * hh;
      auto piece = [&](int key) {
        const T* src = &sh.v[buf][key][cb + 4 * (i & 3)];
        return __builtin_amdgcn_ds_read_tr16_b64_v4i16(
            (__attribute__((address_space(3))) s16x4*)src);
      };
      const s16x4 x0 = piece(kb + i / 4), x1 = piece(kb + 8 + i / 4);
      return __builtin_bit_cast(op_t, __builtin_shufflevector(x0, x1, 0, 1, 2, 3, 4, 5, 6, 7));
    }
  };

  // Scores are scaled by 1/sqrt(d) and, on bf16, kept in the log2 domain of
  // SpRef (fp32 weights do not round, and keep one running maximum).
  constexpr bool kWin = sizeof(T) == 2;
  const float scale = (kWin ? kLog2e : 1.0f) / sqrtf((float)D);
  SpRef rf;
  float& m = rf.ref;
  float l = 0.0f;
  f32x16 acc[C::NCT];
#pragma unroll
  for (int ct = 0; ct < C::NCT; ++ct) acc[ct] = f32x16{};

  TileRegs nx = {}, af = {};
  if (lo < hi) {
    put(fetch(lo), 0);
    if (lo + kTile < hi) nx = fetch(lo + kTile);
  }
  __syncthreads();
  int n = 0;
  for (int j0 = lo; j0 < hi; j0 += kTile, ++n) {
    const int buf = n & 1;
    if (j0 + 2 * kTile < hi) af = fetch(j0 + 2 * kTile);  // tile after next

    f32x16 sc = {};
#pragma unroll
    for (int ks = 0; ks < C::KD; ++ks)
      sc = M::mma(load_op<T>(&sh.k[buf][li][ks * KW + hh * E]), qop[ks], sc);
    // Scaled scores; keys past the range only in the range's last tile
    // (a wave-uniform test, so full tiles carry no masks).
    const bool full = j0 + kTile <= hi;
    float p[16];
    float mt = -INFINITY;
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      p[i] = (full || j0 + row_of(i, hh) < hi) ? sc[i] * scale : -INFINITY;
      mt = fmaxf(mt, p[i]);
    }
    mt = fmaxf(mt, xor32(mt));
    float mn;
    bool moves;
    if constexpr (kWin) {
      moves = rf.take(mt, SpRef::restarts<2>(n), mn);
    } else {
      mn = fmaxf(m, mt);
      moves = __any(mn > m);
    }
    auto ex = [](float x) { return kWin ? __builtin_amdgcn_exp2f(x) : fast_exp(x); };
    float ps = 0.0f;
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      p[i] = as_operand<T>(ex(p[i] - mn));  // exp(-inf) = 0 past the range
      ps += p[i];
    }
    ps += xor32(ps);
    // The accumulators are rescaled only when some query's reference moved:
    // once the maximum settles most tiles skip the 64 multiplies.
    if (moves) {
      const float corr = ex(m - mn);
      l *= corr;
#pragma unroll
      for (int ct = 0; ct < C::NCT; ++ct)
#pragma unroll
        for (int i = 0; i < 16; ++i) acc[ct][i] *= corr;
    }
    l += ps;
    m = mn;
#pragma unroll
    for (int ct = 0; ct < C::NCT; ++ct)
#pragma unroll
      for (int ks = 0; ks < C::KL; ++ks)
        acc[ct] = M::mma(vt_op(buf, ct, ks), cvt_op<T>(&p[ks * E]), acc[ct]);
    if (j0 + kTile < hi) put(nx, buf ^ 1);  // next tile into the free buffer
    nx = af;
    __syncthreads();
  }

  // Partial result of this range: unnormalised O, running max and sum.
  if (li >= L) return;
  if (rg.n == 1) {
    // one range: the result is final, normalised here
    const float inv = 1.0f / l;
    const size_t ob = (((size_t)b * L + li) * Hq + h) * D;
#pragma unroll
    for (int ct = 0; ct < C::NCT; ++ct)
#pragma unroll
      for (int i = 0; i < 16; i += 4) {
        const float o[4] = {acc[ct][i] * inv, acc[ct][i + 1] * inv, acc[ct][i + 2] * inv,
                            acc[ct][i + 3] * inv};
        store_out4<T>(a.out, ob + ct * kTile + row_of(i, hh), o, a.s.out_f32);
      }
    return;
  }
  const size_t row = sp_row(a, r, h, li);
  float* wacc = (float*)a.ws + row * D;
  float* wml = sp_ml<D>(a) + row * 2;
#pragma unroll
  for (int ct = 0; ct < C::NCT; ++ct)
#pragma unroll
    for (int i = 0; i < 16; i += 4)
      *reinterpret_cast<f32x4*>(wacc + ct * kTile + row_of(i, hh)) =
          f32x4{acc[ct][i], acc[ct][i + 1], acc[ct][i + 2], acc[ct][i + 3]};
  if (hh == 0) {
    wml[0] = kWin ? m * 0.6931471805599453f : m;  // (the natural log)
    wml[1] = l;
  }
}


// bf16 with 1, 2, 4 or 8 query heads per KV head: the K and V tiles reach
// LDS by direct global->LDS copies into two rings of R = 4 tile slots, three
// tiles in flight while one is computed, with no registers held for them.
// Each copy instruction reads whole rows, 16 bytes per lane; chunk c of a
// staged K row t sits at position c ^ swz(t), of a V row at c ^ vswz(t), so
// the rows one operand read touches fall in distinct LDS banks (a K operand
// reads one chunk of 32 rows, a transposing V read four chunks of 4 rows per
// half wave).  The slots are distinct arrays and the
// tile loop is unrolled over them, so every copy and every read names its
// slot at compile time.  A wave waits only for its own copies of the tiles it
// is about to read (vmcnt counts the later tiles' copies still in flight),
// then one barrier per tile makes all of them visible and frees the slots the
// next copies reuse.
//
// What bounds the loop is each wave's chain, not the copies: scores (8
// dependent MFMAs), maximum, exponentials, P V (8 MFMAs).  So step n forms
// the scores of tile n + 1 while it takes the softmax of tile n: two
// independent chains whose MFMAs and VALU instructions interleave.  That is
// why K runs one tile ahead of V in its ring.  At 128 requests of 32768 keys:
// 1.72 ms (5.0 TB/s) as one chain, 1.51 ms (5.7 TB/s) so.
template <int D>
struct SpRing {
  static constexpr int EPC = 8;                      // bf16 per 16 bytes
  static constexpr int CPR = D / EPC;                // chunks per row
  static constexpr int RPI = kWave / CPR;            // rows per copy instruction
  static constexpr int RP256 = 256 / (D * 2) > 0 ? 256 / (D * 2) : 1;
  static constexpr int IK = kTile / RPI;             // copies per 32-row tile
  static constexpr int R = 4;                        // ring slots
  __device__ static constexpr int swz(int t) { return (t / RP256) % CPR; }
  __device__ static constexpr int vswz(int t) { return 4 * ((t / RP256) % (CPR / 4)); }
};

// c ? a : b of values: written out over two captured variables it is a choice of
// their addresses, which can leave a lambda's captures in scratch memory.
__device__ inline const bf16* sp_pick(bool c, const bf16* a, const bf16* b) { return c ? a : b; }

template <int D>
struct alignas(16) SpSlot {
  bf16 k[kTile * D];
  bf16 v[kTile * D];
};

template <int D, int NG, bool PAGED>
__global__ __launch_bounds__(kWave* NG, D == 64 && NG == 8 ? 4 : 2) void hyb_sp_ring_kernel(SoftmaxPrefixArgs a, SpCut cut) {
  typedef Mma<bf16> M;
  typedef typename M::op_t op_t;
  typedef SpRing<D> RG;
  constexpr int E = M::E, KW = M::KW, KD = D / KW, KL = kTile / KW, NCT = D / kTile;
  constexpr int EPC = RG::EPC, CPR = RG::CPR, RPI = RG::RPI, IK = RG::IK, R = RG::R;
  constexpr int IPW = 2 * IK / NG;  // copies per wave and step
  static_assert(IPW * NG == 2 * IK, "copies split evenly over the waves");
  static_assert(3 * IPW <= 63, "a wave's copies in flight fit vmcnt");
  __shared__ SpSlot<D> s0, s1, s2, s3;

  const int tid = threadIdx.x, lane = tid & (kWave - 1);
  const int w = __builtin_amdgcn_readfirstlane(tid / kWave);
  const int li = lane & 31, hh = lane >> 5;
  const int Hq = a.s.Hq, Hkv = a.s.Hkv, L = a.s.L, G = Hq / Hkv;
  const int Pmax = a.max_prefix;
  // The KV head varies fastest: the Hkv workgroups that read the same
  // token rows of the cache (each its 1/Hkv share of every row) start
  // together.
  const int g = blockIdx.x % Hkv, r = blockIdx.x / Hkv, h = g * G + w;
  static_assert(sizeof(s3.v) >= kPlanInts * sizeof(int), "the plan's scratch fits a tile");
  const SpRange rg = sp_range(a, sp_plan(a, cut, reinterpret_cast<int*>(s3.v)), r, lane);
  if (rg.b < 0) return;  // uniform: past the plan's last range
  const int b = rg.b, lo = rg.lo, hi = rg.hi;
  const int P = sp_keys(a, b) - L;
  const int ntiles = (hi - lo + kTile - 1) / kTile;
  const size_t qstride = (size_t)Hq * D, kstride = (size_t)Hkv * D;

  op_t qop[KD];
  {
    const bf16* qrow =
        (const bf16*)a.q + ((size_t)b * L * Hq + h) * D + (size_t)min(li, L - 1) * qstride + hh * E;
#pragma unroll
    for (int ks = 0; ks < KD; ++ks) qop[ks] = keep_if<bf16>(li < L, load_op<bf16>(qrow + ks * KW));
  }
  // contiguous: this request's rows; paged: the pool, at KV head g
  const bf16* kc = (const bf16*)a.k_cache + ((PAGED ? 0 : (size_t)b * Pmax * Hkv) + g) * D;
  const bf16* vc = (const bf16*)a.v_cache + ((PAGED ? 0 : (size_t)b * Pmax * Hkv) + g) * D;
  const bf16* kbk = (const bf16*)a.k + ((size_t)b * L * Hkv + g) * D;
  const bf16* vbk = (const bf16*)a.v + ((size_t)b * L * Hkv + g) * D;
  // Paged: the pages of the cached keys of this range, lo .. min(hi, P) - 1,
  // staged in LDS (page index p0 + e at e), clamped to the pool.
  __shared__ int pages[PAGED ? kMaxRangePages : 1];
  const int p0 = lo >> a.page_shift;
  if constexpr (PAGED) {
    const int32_t* ptab = a.page_table + (size_t)b * a.max_pages;
    const int chi = min(hi, P);
    const int np = chi > lo ? ((chi - 1) >> a.page_shift) - p0 + 1 : 0;
    for (int e = tid; e < np; e += kWave * NG) pages[e] = sp_page(a, ptab, (p0 + e) << a.page_shift);
    __syncthreads();
  }

  // Copies of a tile that lies wholly in the cached prefix: a buffer
  // descriptor whose base is the tile's first row (a scalar) and, per lane
  // and copy, the 32-bit offset of its 16-byte piece, which is the same for
  // every tile.  Tiles that reach past the cache or the range take the
  // general path below.  Copy ins of a step is K's (kv = 0) or V's (kv = 1);
  // a wave's copies are all of one kind, except with one wave (NG = 1).
  int voff[IPW];
#pragma unroll
  for (int u = 0; u < IPW; ++u) {
    const int ins = w * IPW + u, i = ins % IK;
    const int t = i * RPI + lane / CPR, pos = lane % CPR;
    const int sw = ins < IK ? RG::swz(t) : RG::vswz(t);
    voff[u] = (int)(((size_t)t * kstride + (size_t)((pos ^ sw) * EPC)) * sizeof(bf16));
  }
  const int cend = min(hi, P);  // keys below this come from the cache
  // The order of the tiles.  Those that reach past the cache (the range's last
  // one or two, nlate of them: a block is at most a tile long) come first, the last
  // one foremost: their copies are all issued before the loop, and only tile 0
  // can be partial, so the loop's steps need neither the general copies nor
  // masks.  (With them last and a second set of steps for the last tiles the
  // code was twice as long, and a short range, which runs it once, waited for its
  // instructions: with one head per KV head at d = 128 one request of 300 keys
  // took 21.4 us, now 15.7, 32 of 512 28.1 and 24.1, 32 of 4096 138 and 115.)
  const int nlate = ntiles - (cend > lo ? (cend - lo) / kTile : 0);
  auto first_key = [&](int n) __attribute__((always_inline)) {
    return lo + (n < nlate ? ntiles - 1 - n : n - nlate) * kTile;
  };
  constexpr int NKV = NG == 1 ? 2 : 1;      // kinds of copies per wave
  constexpr int IPK = IPW / NKV;            // copies per kind
  // This wave's copies u0 .. u0 + IPK - 1, of kind kv, of tile n into dst.
  auto issue_cached = [&](int kv, int u0, int n, bf16* dst) __attribute__((always_inline)) {
    const int j0 = lo + (n - nlate) * kTile;
    const bf16* cb = sp_pick(kv == 0, kc, vc);
    if constexpr (PAGED) {
      const int pi = j0 >> a.page_shift;
      cb += ((ptrdiff_t)__builtin_amdgcn_readfirstlane(pages[pi - p0]) - pi) *
            ((ptrdiff_t)kstride << a.page_shift);
    }
    cb += (size_t)j0 * kstride;
    const int span = (int)((size_t)kTile * kstride * sizeof(bf16));
    const __amdgpu_buffer_rsrc_t rs =
        __builtin_amdgcn_make_buffer_rsrc(const_cast<bf16*>(cb), 0, span, kBufferWord3);
#pragma unroll
    for (int u = u0; u < u0 + IPK; ++u) buf_to_lds16(rs, dst + (w * IPW + u) % IK * RPI * D, voff[u], 0);
  };
  // The same of a tile that reaches past the cache (keys past the range read
  // the range's last key, in bounds, and are masked below).
  auto issue_general = [&](int kv, int u0, int n, bf16* dst) __attribute__((always_inline)) {
    const int j0 = first_key(n);
    const bf16* cb = sp_pick(kv == 0, kc, vc);
    if constexpr (PAGED) {
      // the tile's rows (clamped to the range, all >= j0) lie in the page of
      // row j0: that page's base, shifted so that base + j * kstride is row j
      if (j0 < P) {
        const int pi = j0 >> a.page_shift;
        cb += ((ptrdiff_t)pages[pi - p0] - pi) * ((ptrdiff_t)kstride << a.page_shift);
      }
    }
    const bf16* blk = sp_pick(kv == 0, kbk, vbk);
#pragma unroll
    for (int u = u0; u < u0 + IPK; ++u) {
      const int i = (w * IPW + u) % IK;
      const int t = i * RPI + lane / CPR, pos = lane % CPR;
      const int j = min(j0 + t, hi - 1);
      const bf16* row = sp_pick(j < P, cb, blk) + (size_t)(j < P ? j : j - P) * kstride;
      __builtin_amdgcn_global_load_lds(
          (const __attribute__((address_space(1))) void*)(row + (pos ^ (kv == 0 ? RG::swz(t) : RG::vswz(t))) * EPC),
          (__attribute__((address_space(3))) void*)(dst + i * RPI * D), 16, 0, 0);
    }
  };
  // The copies of step n: K of tile nk and V of tile nv, where they exist
  // (early: tiles 0 and 1, which may reach past the cache).
  auto issue = [&](auto early, int nk, SpSlot<D>& sk, int nv, SpSlot<D>& sv) __attribute__((always_inline)) {
    auto one = [&](int kv, int u0, int n, bf16* dst) __attribute__((always_inline)) {
      if constexpr (decltype(early)::value) {
        if (n < nlate) {
          issue_general(kv, u0, n, dst);
          return;
        }
      }
      issue_cached(kv, u0, n, dst);
    };
    if constexpr (NG == 1) {
      if (nk < ntiles) one(0, 0, nk, sk.k);
      if (nv >= 0 && nv < ntiles) one(1, IPK, nv, sv.v);
    } else {
      const int kv = w * IPW / IK, n = kv == 0 ? nk : nv;
      if (n >= 0 && n < ntiles) one(kv, 0, n, kv == 0 ? sk.k : sv.v);
    }
  };

  // Scores and the reference m (SpRef) are kept in the log2 domain (scaled by
  // log2 e with 1/sqrt(d)), so each weight is one fma and one exp2;
  // m is converted back where it is written out for the combine.
  const float scale = 1.4426950408889634f / sqrtf((float)D);
  // The running sum of the weights comes from the MFMAs, so it is the sum of
  // the same rounded weights that enter P V: a 16x16 product whose column
  // li % 16 holds, as its contraction quarters, the keys of queries li % 16
  // (even quarters) and li % 16 + 16 (odd ones).  Row x of the left operand
  // is one on the quarters of the parity of x / 4, which is that of the lane
  // that receives the row, so register 0 is the sum of the lane's own query
  // (only that register is kept rescaled).
  SpRef rf;
  float& m = rf.ref;
  f32x16 acc[NCT];
  f32x4 lsum = {};
#pragma unroll
  for (int ct = 0; ct < NCT; ++ct) acc[ct] = f32x16{};
  op_t ones;
#pragma unroll
  for (int e = 0; e < E; ++e) ones[e] = (bf16)(((lane >> 4) ^ (lane >> 2)) & 1 ? 0.0f : 1.0f);

  // Raw scores of a tile: keys in rows, queries in columns.
  auto k_op = [&](const bf16* kt, int ks) __attribute__((always_inline)) -> op_t {
    const int c = 2 * ks + hh;  // 16-byte chunk of elements ks*KW + hh*E
    return load_op<bf16>(&kt[li * D + (c ^ RG::swz(li)) * EPC]);
  };
  // Scores of the tile of the current step, already in the reference (and the
  // accumulators rescaled to it).
  f32x16 sc;
  // Takes the scores of tile n into sc and the reference.  The accumulators are
  // rescaled only when some query's reference moved: once the maximum settles
  // most tiles skip the 64 multiplies.  Keys past the range, in tile 0 only,
  // are masked.
  auto take_scores = [&](auto check, int n, const f32x16& s) __attribute__((always_inline)) {
    sc = s;
    if constexpr (decltype(check)::value) {
      const int j0 = first_key(n);
      if (j0 + kTile > hi) {  // uniform
#pragma unroll
        for (int i = 0; i < 16; ++i) sc[i] = j0 + row_of(i, hh) < hi ? sc[i] : -INFINITY;
      }
    }
    float mt = sc[0];
#pragma unroll
    for (int i = 1; i < 16; ++i) mt = fmaxf(mt, sc[i]);
    mt = fmaxf(mt, xor32(mt));
    float mn;
    if (rf.take(mt * scale, SpRef::restarts<1>(n), mn)) {
      const float corr = __builtin_amdgcn_exp2f(m - mn);
      lsum[0] *= corr;
#pragma unroll
      for (int ct = 0; ct < NCT; ++ct)
#pragma unroll
        for (int i = 0; i < 16; ++i) acc[ct][i] *= corr;
    }
    m = mn;
  };

  // Weights and P V of tile n (its scores in sc, its V in vt) and the scores
  // of tile n + 1 (its K in kt; not with LAST), then that tile's maximum.
  auto compute = [&](auto last, int n, const bf16* kt, const bf16* vt) __attribute__((always_inline)) {
    constexpr bool LAST = decltype(last)::value;
    op_t kop[KD];
    if constexpr (!LAST) {
#pragma unroll
      for (int ks = 0; ks < KD; ++ks) kop[ks] = k_op(kt, ks);
    }
    f32x16 sn = {};
    if constexpr (!LAST) {
#pragma unroll
      for (int ks = 0; ks < KD; ++ks) sn = M::mma(kop[ks], qop[ks], sn);
    }
    float p[16];
#pragma unroll
    for (int i = 0; i < 16; ++i) p[i] = __builtin_amdgcn_exp2f(__builtin_fmaf(sc[i], scale, -m));
    op_t pop[KL];
#pragma unroll
    for (int ks = 0; ks < KL; ++ks) pop[ks] = cvt_op<bf16>(&p[ks * E]);
    // V^T operands by transposing reads: in each 16-lane quarter lane i
    // addresses key kb + i/4 at columns cb + 4*(i%4) .. +3 and receives
    // keys kb .. kb+3 of column cb + i.
    typedef short s16x4 __attribute__((ext_vector_type(4)));
    const int qi = lane & 15;
    op_t vop[NCT][KL];
#pragma unroll
    for (int ct = 0; ct < NCT; ++ct) {
      const int col = ct * kTile + 16 * ((lane >> 4) & 1) + 4 * (qi & 3);
#pragma unroll
      for (int ks = 0; ks < KL; ++ks) {
        auto piece = [&](int t) {
          // (t = kb + 8n: vswz(t) is that of the lane's qi / 4)
          const bf16* src = &vt[t * D + ((col / EPC) ^ RG::vswz(qi / 4)) * EPC + col % EPC];
          return __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4*)src);
        };
        const int kb = 16 * ks + 4 * hh + qi / 4;
        const s16x4 x0 = piece(kb), x1 = piece(kb + 8);
        vop[ct][ks] = __builtin_bit_cast(op_t, __builtin_shufflevector(x0, x1, 0, 1, 2, 3, 4, 5, 6, 7));
      }
    }
#pragma unroll
    for (int ct = 0; ct < NCT; ++ct)
#pragma unroll
      for (int ks = 0; ks < KL; ++ks) acc[ct] = M::mma(vop[ct][ks], pop[ks], acc[ct]);
#pragma unroll
    for (int ks = 0; ks < KL; ++ks) lsum = Mma16<bf16>::mma(ones, pop[ks], lsum);
    if constexpr (!LAST) {
      // The order of issue: K's operands; the score MFMAs with the weights
      // between them, V's operands requested behind the first half of them;
      // then P V with the next tile's maximum.
      __builtin_amdgcn_sched_group_barrier(0x100, KD, 0);  // LDS reads
#pragma unroll
      for (int ks = 0; ks < KD / 2; ++ks) {
        __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);  // an MFMA
        __builtin_amdgcn_sched_group_barrier(0x402, 6, 0);  // VALU, exp
      }
#pragma unroll
      for (int ks = KD / 2; ks < KD; ++ks) {
        __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
        __builtin_amdgcn_sched_group_barrier(0x100, 4 * NCT * KL / KD, 0);
        __builtin_amdgcn_sched_group_barrier(0x402, 6, 0);
      }
      take_scores(std::false_type{}, n + 1, sn);
    }
  };

  // Wait for this wave's copies of the tiles of a step, with at most `later`
  // steps' copies issued after them still in flight.
  auto wait_step = [&](int later) __attribute__((always_inline)) {
    if (later >= 3) asm volatile("s_waitcnt vmcnt(%0)" ::"n"(3 * IPW) : "memory");
    else if (later == 2) asm volatile("s_waitcnt vmcnt(%0)" ::"n"(2 * IPW) : "memory");
    else if (later == 1) asm volatile("s_waitcnt vmcnt(%0)" ::"n"(IPW) : "memory");
    else asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  };
  auto slot = [&](auto S) -> SpSlot<D>& {
    if constexpr (decltype(S)::value == 0) return s0;
    else if constexpr (decltype(S)::value == 1) return s1;
    else if constexpr (decltype(S)::value == 2) return s2;
    else return s3;
  };
  // A wave's last tile whose copies it must see: V's wave n, K's wave n + 1.
  // With one wave, a step's copies are K n + 1 and V n; whole steps are
  // counted while both kinds are still issued.
  const int ahead = NG == 1 || w * IPW / IK == 0 ? 1 : 0;
  auto step = [&](int n, auto S) __attribute__((always_inline)) {
    constexpr int SV = decltype(S)::value;
    const int later = ntiles - 1 - n - ahead;
    if constexpr (NG == 1) wait_step(later >= 2 ? 2 : 0);
    else wait_step(min(2, later));
    lds_barrier_nodrain();  // K n+1 and V n visible everywhere; K n's and V n-1's slots free
    issue(std::false_type{}, n + R, slot(S), n + R - 1, slot(std::integral_constant<int, (SV + R - 1) % R>{}));
    compute(std::false_type{}, n, slot(std::integral_constant<int, (SV + 1) % R>{}).k, slot(S).v);
  };

  // Copies of K 0 .. R-1 and V 0 .. R-2, in the order of the steps' copies.
  const std::true_type yes{};
  issue(yes, 0, s0, -1, s0);
  issue(yes, 1, s1, 0, s0);
  issue(yes, 2, s2, 1, s1);  // (K of tile 2 is a cached tile's)
  issue(std::false_type{}, 3, s3, 2, s2);
  if constexpr (NG == 1) wait_step(ntiles >= R ? 3 : 0);
  else wait_step(ahead ? min(3, ntiles - 1) : 3);  // (V's waves need nothing yet)
  lds_barrier_nodrain();
  {
    f32x16 s = {};
#pragma unroll
    for (int ks = 0; ks < KD; ++ks) s = M::mma(k_op(s0.k, ks), qop[ks], s);
    take_scores(yes, 0, s);
  }
  int n = 0;
  for (; n + R < ntiles; n += R) {
    step(n, std::integral_constant<int, 0>{});
    step(n + 1, std::integral_constant<int, 1>{});
    step(n + 2, std::integral_constant<int, 2>{});
    step(n + 3, std::integral_constant<int, 3>{});
  }
  if (n + 1 < ntiles) step(n, std::integral_constant<int, 0>{});
  if (n + 2 < ntiles) step(n + 1, std::integral_constant<int, 1>{});
  if (n + 3 < ntiles) step(n + 2, std::integral_constant<int, 2>{});
  // the last tile: every copy has landed
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  lds_barrier_nodrain();
  const int rest = ntiles - n;  // 1 .. R
  compute(yes, ntiles - 1, nullptr, rest == 2 ? s1.v : rest == 3 ? s2.v : rest == 4 ? s3.v : s0.v);

  if (li >= L) return;
  const float l = lsum[0];
  if (rg.n == 1) {
    // one range: the result is final, normalised here
    const float inv = 1.0f / l;
    const size_t ob = (((size_t)b * L + li) * Hq + h) * D;
#pragma unroll
    for (int ct = 0; ct < NCT; ++ct)
#pragma unroll
      for (int i = 0; i < 16; i += 4) {
        const float o[4] = {acc[ct][i] * inv, acc[ct][i + 1] * inv, acc[ct][i + 2] * inv,
                            acc[ct][i + 3] * inv};
        store_out4<bf16>(a.out, ob + ct * kTile + row_of(i, hh), o, a.s.out_f32);
      }
    return;
  }
  const size_t row = sp_row(a, r, h, li);
  float* wacc = (float*)a.ws + row * D;
  float* wml = sp_ml<D>(a) + row * 2;
#pragma unroll
  for (int ct = 0; ct < NCT; ++ct)
#pragma unroll
    for (int i = 0; i < 16; i += 4)
      *reinterpret_cast<f32x4*>(wacc + ct * kTile + row_of(i, hh)) =
          f32x4{acc[ct][i], acc[ct][i + 1], acc[ct][i + 2], acc[ct][i + 3]};
  if (hh == 0) {
    wml[0] = m * 0.6931471805599453f;  // back to the natural log
    wml[1] = l;
  }
}

// Merge of the partial results of the requests that have several ranges.  A
// workgroup's unit of work is RPB rows of a (request, head), a thread 4
// columns of a row (16-byte loads); loads of several ranges are in flight at
// once, and up to four ranges are read before their weights are known.  A
// small merge is a chain of latencies (the plan, the maxima, the rows), so as
// many workgroups run as the chip holds (2048) and most take one unit: 32
// requests of 1024 keys 12.3 us, where 1024 workgroups of two units with
// the rows requested after the maxima took 13.7 us (8 requests: 7.2, now
// 5.4).
template <typename T, int D>
__global__ __launch_bounds__(256) void hyb_sp_combine_kernel(SoftmaxPrefixArgs a, SpCut cut) {
  constexpr int TPR = D / 4;              // threads per row
  constexpr int RPB = 256 / TPR;          // rows per unit
  __shared__ alignas(16) int plan[kPlanInts];
  const SpPlan p = sp_plan(a, cut, plan);
  if (p.whole) return;  // every row is already written out
  const int Hq = a.s.Hq, L = a.s.L, lane = threadIdx.x & (kWave - 1);
  const int upb = (L + RPB - 1) / RPB;    // units of a (request, head)
  const float* wacc = (const float*)a.ws;
  const float* wml = sp_ml<D>(a);
  const size_t step = (size_t)Hq * L;  // rows from one range to the next
  for (int u = blockIdx.x; u < a.s.B * Hq * upb; u += gridDim.x) {
    const int bh = u / upb, b = bh / Hq, h = bh % Hq;
    const int n = sp_ranges(p, sp_tiles(a, b));
    if (n == 1) continue;  // uniform: already written out
    int base = 0;
    for (int b0 = lane; b0 < b; b0 += kWave) base += sp_ranges(p, sp_tiles(a, b0));
    base = wave_all(base, AddOp{});
    const int i = u % upb * RPB + threadIdx.x / TPR, c = (threadIdx.x % TPR) * 4;
    if (i >= L) continue;  // (no barrier or exchange follows in this unit)
    const size_t row0 = sp_row(a, base, h, i);
    float M = -INFINITY;
    f32x4 num = {0.0f, 0.0f, 0.0f, 0.0f};
    float den = 0.0f;
    if (n <= 4) {
      float2 ml[4];
      f32x4 x[4];
#pragma unroll
      for (int s = 0; s < 4; ++s) {
        const size_t rr = row0 + min(s, n - 1) * step;
        ml[s] = *reinterpret_cast<const float2*>(wml + rr * 2);
        x[s] = *reinterpret_cast<const f32x4*>(wacc + rr * D + c);
      }
#pragma unroll
      for (int s = 0; s < 4; ++s) M = fmaxf(M, ml[s].x);
#pragma unroll
      for (int s = 0; s < 4; ++s) {
        if (s >= n || ml[s].x == -INFINITY) continue;
        const float wgt = expf(ml[s].x - M);
#pragma unroll
        for (int e = 0; e < 4; ++e) num[e] += wgt * x[s][e];
        den += wgt * ml[s].y;
      }
    } else {
#pragma unroll 8
      for (int s = 0; s < n; ++s) M = fmaxf(M, wml[(row0 + s * step) * 2]);
#pragma unroll 4
      for (int s = 0; s < n; ++s) {
        const size_t rr = row0 + s * step;
        const float ms = wml[rr * 2];
        if (ms == -INFINITY) continue;  // every score of the range is -inf
        const float wgt = expf(ms - M);
        const f32x4 x = *reinterpret_cast<const f32x4*>(wacc + rr * D + c);
#pragma unroll
        for (int e = 0; e < 4; ++e) num[e] += wgt * x[e];
        den += wgt * wml[rr * 2 + 1];
      }
    }
    const float o[4] = {num[0] / den, num[1] / den, num[2] / den, num[3] / den};
    store_out4<T>(a.out, (((size_t)b * L + i) * Hq + h) * D + c, o, a.s.out_f32);
  }
}

// Ranges per request on average at most (the workspace and the grid hold
// that many): about 2048 workgroups of ranges of at least 512 keys.
int softmax_prefix_splits(const Shape& s, int max_prefix) {
  const long units = (long)s.B * s.Hkv;
  long want = units > 0 ? (2048 + units - 1) / units : 1;
  const long cap = ((long)max_prefix + s.L + 511) / 512;
  if (want > cap) want = cap;
  // no range longer than kMaxRange keys (the paged kernel stages a range's
  // page numbers in LDS)
  const long least = ((long)max_prefix + s.L + kMaxRange - 1) / kMaxRange;
  if (want < least) want = least;
  if (want < 1) want = 1;
  return (int)want;
}

// A single KV range per (request, KV head) writes the normalised output
// directly and needs no workspace.
size_t softmax_prefix_ws_bytes(const Shape& s, int n_split) {
  if (n_split <= 1) return 0;
  return (size_t)s.B * s.Hq * n_split * s.L * (s.D + 2) * sizeof(float);
}

// Workgroups of a range kernel that the chip holds at once, by its LDS and
// registers as built.  Waves go to the four SIMDs in turn: 3, 5, 6 and 7 of them
// are counted as the next multiple of four (the odd ones seldom fit in between).
template <typename K>
static int sp_resident(K kernel, int waves) {
  int n = 0;
  const int w = waves <= 2 ? waves : (waves + 3) / 4 * 4;
  const hipError_t e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, kernel, kWave * w, 0);
  return 256 * (e == hipSuccess ? max(1, n) : 1);
}

template <typename K>
static hipError_t sp_launch(K kernel, int resident, int waves, bool ring, const SoftmaxPrefixArgs& a, hipStream_t st,
                            SpCut* out) {
  const int ns = a.n_split;
  SpCut cut;
  // Of the ring's workgroups two per CU, one with more than four waves, keep
  // the memory as busy as more do, three tiles of each in flight; the
  // register-staged kernel is bound by its waves' own chains.  (Two, or one, for
  // every kernel, also as what the chip holds, was right at d = 128 only: at
  // d = 64 up to five of the ring's workgroups fit: 32 requests of 1024 keys, 8
  // KV heads of one head, 26.7 us, now 19.2; 32 of 1 to 4096 keys at 16 KV heads,
  // paged, 115 and 77.)
  cut.slots = max(1, (waves > 4 ? min(resident, 256) : resident) / a.s.Hkv);
  cut.sat = ring ? max(1, min(cut.slots, (waves > 4 ? 256 : 512) / a.s.Hkv)) : cut.slots;
  // Ranges of a plan at most: three rounds, within the workspace, and at
  // least what the longest range allows.
  const int need = (int)(((long)a.max_prefix + a.s.L + kMaxRange - 1) / kMaxRange);
  cut.limit = min(a.s.B * ns, max(a.s.B * need, 3 * cut.sat));
  cut.layer = max(1, 256 / a.s.Hkv);
  // Where ranges of at most 512 keys of full-length requests fit one round,
  // the host cuts every request into those: there is little to gain from the
  // lengths, and working a plan out costs each kernel a few us (32 requests of
  // 1024 keys 43.8 against 37.4 us so, 8 of 4096 43.5 and 39.4, one of 8192
  // 32.7 and 28.8).
  const int tmax = (int)(((long)a.max_prefix + a.s.L + kTile - 1) / kTile);
  const int even = (tmax + ns - 1) / ns;
  cut.c = 0;
  if ((long)a.s.B * ns <= cut.slots && even <= 16) {
    cut.c = even;
    cut.limit = a.s.B * ns;  // (full-length requests' ranges)
  }
  *out = cut;
  hipLaunchKernelGGL(kernel, dim3(a.s.Hkv * cut.limit), dim3(kWave * waves), 0, st, a, cut);
  return hipGetLastError();
}

template <typename T, int D, bool PAGED>
static hipError_t sp_go(const SoftmaxPrefixArgs& a, hipStream_t st) {
  SpCut cut;
  hipError_t e;
  // (a paged cache is cut as the contiguous one is, for the same bits: by what fits
  // of both their kernels)
#define HYB_SP_CASE(NG, RING, ...)                                              \
  case NG: {                                                                    \
    static const int resident =                                                 \
        min(sp_resident(__VA_ARGS__, true>, NG), sp_resident(__VA_ARGS__, false>, NG)); \
    e = sp_launch(__VA_ARGS__, PAGED>, resident, NG, RING, a, st, &cut);        \
    break;                                                                      \
  }
  // bf16 with 1, 2, 4 or 8 query heads per KV head: the copy ring; else the
  // register-staged kernel.
  if constexpr (sizeof(T) == 2) {
    switch (a.s.Hq / a.s.Hkv) {
      HYB_SP_CASE(1, true, hyb_sp_ring_kernel<D, 1)
      HYB_SP_CASE(2, true, hyb_sp_ring_kernel<D, 2)
      HYB_SP_CASE(3, false, hyb_sp_partial_kernel<T, D, 3)
      HYB_SP_CASE(4, true, hyb_sp_ring_kernel<D, 4)
      HYB_SP_CASE(5, false, hyb_sp_partial_kernel<T, D, 5)
      HYB_SP_CASE(6, false, hyb_sp_partial_kernel<T, D, 6)
      HYB_SP_CASE(7, false, hyb_sp_partial_kernel<T, D, 7)
      HYB_SP_CASE(8, true, hyb_sp_ring_kernel<D, 8)
      default: return hipErrorInvalidValue;
    }
  } else {
    switch (a.s.Hq / a.s.Hkv) {
      HYB_SP_CASE(1, false, hyb_sp_partial_kernel<T, D, 1)
      HYB_SP_CASE(2, false, hyb_sp_partial_kernel<T, D, 2)
      HYB_SP_CASE(3, false, hyb_sp_partial_kernel<T, D, 3)
      HYB_SP_CASE(4, false, hyb_sp_partial_kernel<T, D, 4)
      HYB_SP_CASE(5, false, hyb_sp_partial_kernel<T, D, 5)
      HYB_SP_CASE(6, false, hyb_sp_partial_kernel<T, D, 6)
      HYB_SP_CASE(7, false, hyb_sp_partial_kernel<T, D, 7)
      HYB_SP_CASE(8, false, hyb_sp_partial_kernel<T, D, 8)
      default: return hipErrorInvalidValue;
    }
  }
#undef HYB_SP_CASE
  if (e != hipSuccess || a.n_split == 1) return e;  // one range: already written out
  const long units = (long)a.s.B * a.s.Hq * ((a.s.L + 1024 / D - 1) / (1024 / D));
  hipLaunchKernelGGL((hyb_sp_combine_kernel<T, D>), dim3((unsigned)std::min<long>(units, 2048)), dim3(256), 0, st,
                     a, cut);
  return hipGetLastError();
}

template <bool PAGED>
static hipError_t sp_dispatch(const SoftmaxPrefixArgs& a, hipStream_t st) {
  if (a.s.dtype == 1)
    return a.s.D == 64 ? sp_go<bf16, 64, PAGED>(a, st) : sp_go<bf16, 128, PAGED>(a, st);
  return a.s.D == 64 ? sp_go<float, 64, PAGED>(a, st) : sp_go<float, 128, PAGED>(a, st);
}

hipError_t launch_softmax_prefix(const SoftmaxPrefixArgs& a, hipStream_t st) {
  if (a.s.Hq / a.s.Hkv > kMaxGroup) return hipErrorInvalidValue;
  if (a.page_table) {
    if (a.page_shift < 5 || a.n_pages < 1) return hipErrorInvalidValue;
    return sp_dispatch<true>(a, st);
  }
  return sp_dispatch<false>(a, st);
}

}  // namespace hyb
