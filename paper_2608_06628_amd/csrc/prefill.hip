// prefill.hip -- block-causal prefill of a prompt into the recurrent state
// (Figure 2 pattern): block c is answered against the state of blocks
// 0..c-1 -- exact softmax inside the block, linear readout of the state,
// gated merge (Section 3.1) -- and is then committed,
// S += phi(K_c)^T V_c, z += sum phi(K_c).
//
// Sequence segments.  The prompt's blocks are cut into nseg segments so that
// the grid fills the chip (SegPlan).  A first launch (delta mode) computes the
// state increments dS = sum_c phi(K_c)^T V_c and dz of the blocks of segments
// 0 .. nseg-2, in pieces of a segment each or smaller, into the caller's
// workspace; a second (the scan) turns them into each segment's starting
// state, S + the increments of the pieces before it; the third (walk mode)
// walks each segment's blocks from there as below, and the last segment
// writes the final state.  Only the associativity of the sum is used, so the
// result is the sequential one up to rounding order.  Without outputs no
// segment walks: the pieces cover the whole prompt and the scan adds them to
// S.
// Ordering: with nseg > 1 the walk segments start from what the scan left in
// the workspace, never from S, z themselves, which the last segment
// overwrites in the same launch (workgroups of one launch are not ordered).
//
// Within a segment, one workgroup per (request b, query head h) walks the
// blocks in order, with the next block's Q, K and V in flight while the
// current one is computed.
// Wave w of NW = D/32 keeps state columns 32w .. 32w+31 of all f rows in fp32
// MFMA accumulators for the whole prompt, so the state is read from HBM once
// and written once.  The accumulator tile doubles as the A operand of the
// readout O_lin^T = S^T phi(Q)^T: register j of the flattened tile is
// contraction element j % E of k-step j / E, i.e. state row
// r = 32*(j/16) + row_of(j%16, hh), and phi(Q) is read from LDS in that
// order.  Block tokens enter every product in the accumulator order of the
// score tile (token row_of(ks*E+e, hh)), so one set of V registers serves
// both P V and the commit.  As in the commit kernel, phi(K) enters the state
// update as a bf16 pair hi + lo on the bf16 path.
#include <type_traits>

#include "device.h"
#include "featmap.h"
#include "launch.h"

namespace hyb {

template <typename T, int D, int F>
struct PrefillCfg {
  typedef Mma<T> M;
  typedef typename M::op_t op_t;
  static constexpr int NW = D / kTile;
  static constexpr int f = 2 * F;
  static constexpr int NRT = f / kTile;
  static constexpr int KD = D / M::KW;
  static constexpr int KF = f / M::KW;
  static constexpr int KL = kTile / M::KW;
  static constexpr int PHI_LD = f + 16 / (int)sizeof(T);
  static constexpr int PT_LD = kTile + 16 / (int)sizeof(T);
  static constexpr int NPART = sizeof(T) == 2 ? 2 : 1;  // hi (+ lo) parts
  typedef FeatMap<T, D, F, NW> FM;
  struct alignas(16) Smem {
    T phiQ[kTile][PHI_LD];         // phi(q_i)[r] at [i][r]
    T phiKT[NPART][f][PT_LD];      // phi(k_t)[r] at [part][r][t]
    float z[f];
    float lden[NW][kTile];         // per-wave partial phi(q_i) . z
    typename FM::Smem fq, fk;
  };
};

// Workspace layout (nseg > 1): the increments dS [units][npieces][D][f] and
// dz [units][npieces][f], then the incoming state, S0 [units][D][f] and
// z0 [units][f].  The scan replaces the increment of piece s * ppseg - 1 by
// the starting state of segment s = 1 .. nseg-1.
__device__ inline float* prefill_start_S(const PrefillArgs& a, const SegPlan& p, int u, int seg) {
  const size_t f = 2 * (size_t)a.s.F, units = (size_t)a.s.B * a.s.Hq, npc = p.npieces();
  const size_t at = seg > 0 ? (size_t)u * npc + seg * p.ppseg - 1 : 0;
  return seg > 0 ? a.ws + at * a.s.D * f
                 : a.ws + units * npc * (a.s.D * f + f) + (size_t)u * a.s.D * f;
}
__device__ inline float* prefill_start_z(const PrefillArgs& a, const SegPlan& p, int u, int seg) {
  const size_t f = 2 * (size_t)a.s.F, units = (size_t)a.s.B * a.s.Hq, npc = p.npieces();
  const size_t at = seg > 0 ? (size_t)u * npc + seg * p.ppseg - 1 : 0;
  return seg > 0 ? a.ws + units * npc * a.s.D * f + at * f
                 : a.ws + units * npc * (a.s.D * f + f) + units * a.s.D * f + (size_t)u * f;
}

// The scan over the pieces of every (request, head) unit: a thread takes four
// consecutive floats of the state (or of z) through all segments, so every
// load of it is independent of the sums and several are in flight.  FINAL: no
// segment walks; S, z + all pieces go back to S, z.  A unit whose slot is out
// of range is skipped (its walk reads no starting state).
// Bound by its bytes (64 KiB per unit, piece and segment at d = f = 128).  As
// a pass of its own it costs 10 us at 8 x 8192 tokens (16.9 MB of increments,
// 42 MB read and written), where copying S and summing the pieces at each walk's start cost 12 us and
// a chain of loads per segment; that chain kept a prompt to 8 segments.
template <bool FINAL>
__global__ __launch_bounds__(256) void hyb_prefill_scan_kernel(PrefillArgs a, SegPlan p) {
  const int Hq = a.s.Hq;
  const size_t f = 2 * (size_t)a.s.F, n = (size_t)a.s.D * f, per = (n + f) / 4;
  const int wpu = (int)((per + blockDim.x - 1) / blockDim.x);  // workgroups per unit
  const int u = blockIdx.x / wpu, b = u / Hq, h = u % Hq;
  const int slot = a.slots ? a.slots[b] : b;
  if (slot < 0 || slot >= a.s.n_slots) return;
  const size_t i = (size_t)(blockIdx.x % wpu) * blockDim.x + threadIdx.x;
  if (i >= per) return;
  const bool isz = i >= n / 4;
  const size_t e = isz ? i * 4 - n : i * 4, len = isz ? f : n;
  const size_t units = (size_t)a.s.B * Hq, npc = p.npieces(), sbase = (size_t)slot * Hq + h;
  float* st = (isz ? a.z + sbase * f : a.S + sbase * n) + e;
  float* inc = (isz ? a.ws + units * npc * n : a.ws) + (size_t)u * npc * len + e;
  f32x4 acc = *reinterpret_cast<const f32x4*>(st);
  if constexpr (FINAL) {
#pragma unroll 8
    for (int pc = 0; pc < p.npieces(); ++pc) acc += *reinterpret_cast<const f32x4*>(inc + pc * len);
    *reinterpret_cast<f32x4*>(st) = acc;
  } else {
    *reinterpret_cast<f32x4*>((isz ? prefill_start_z(a, p, u, 0) : prefill_start_S(a, p, u, 0)) + e) = acc;
    // (a piece is read before the start that replaces it is written)
    constexpr int A = 8;  // pieces in flight
    f32x4 x[A];
    for (int p0 = 0; p0 < p.npieces(); p0 += A) {
#pragma unroll
      for (int j = 0; j < A; ++j)
        x[j] = *reinterpret_cast<const f32x4*>(inc + min(p0 + j, p.npieces() - 1) * len);
#pragma unroll
      for (int j = 0; j < A; ++j) {
        const int pc = p0 + j;
        if (pc >= p.npieces()) break;
        acc += x[j];
        if ((pc + 1) % p.ppseg == 0) *reinterpret_cast<f32x4*>(inc + pc * len) = acc;
      }
    }
  }
}

template <typename T, int D, int F>
__global__ __launch_bounds__(kWave*(D / kTile)) void hyb_prefill_kernel(
    PrefillArgs a, SegPlan p, int delta) {
  typedef PrefillCfg<T, D, F> C;
  typedef typename C::M M;
  typedef typename C::op_t op_t;
  typedef typename C::FM FM;
  constexpr int f = C::f, E = M::E, KW = M::KW;
  __shared__ typename C::Smem sh;

  const int tid = threadIdx.x, lane = tid & (kWave - 1), w = tid / kWave;
  const int li = lane & 31, hh = lane >> 5;
  const int Hq = a.s.Hq, Hkv = a.s.Hkv, L = a.s.L, T_ = a.T;
  // Unit u = (b, h) varies fastest, so the heads of one KV group and segment
  // are neighbours (on one XCD) and share K and V in L2.
  // (delta mode: one workgroup per (unit, piece); walk mode: per (unit,
  // segment))
  const int units = a.s.B * Hq, nseg = p.nseg, npc = p.npieces();
  const int vix = xcd_unit(blockIdx.x, units * (delta ? npc : nseg));
  const int u = vix % units, seg = vix / units;
  const int b = u / Hq, h = u % Hq, g = h / (Hq / Hkv);
  const int slot = a.slots ? a.slots[b] : b;
  const bool want_out = !delta && a.out != nullptr;  // (no outputs: nseg = 1)
  const bool last = !delta && seg == nseg - 1;
  const size_t qstride = (size_t)Hq * D, kstride = (size_t)Hkv * D;
  const int col = w * kTile + li;
  const int nblk = T_ / L;
  const int blk0 = delta ? p.piece_lo(seg) : seg * p.sb;
  const int blk1 = min(nblk, delta ? p.piece_hi(seg) : blk0 + p.sb);
  if (slot < 0 || slot >= a.s.n_slots) {  // uniform per workgroup
    if (want_out) {
      const size_t ob = ((size_t)b * T_ * Hq + h) * D;
      for (int t = blk0 * L; t < blk1 * L; ++t)
        for (int c = tid; c < D; c += blockDim.x)
          store_out1<T>(a.out, ob + (size_t)t * qstride + c, __builtin_nanf(""),
                        a.s.out_f32);
    }
    return;
  }
  const size_t sbase = (size_t)slot * Hq + h;
  float* __restrict__ Sh = a.S + sbase * f * D;
  float* __restrict__ zh = a.z + sbase * f;
  // Workspace: dS [units][npieces][D][f] (transposed, as S), then dz
  // [units][npieces][f].
  float* __restrict__ wsS = a.ws + (size_t)u * npc * D * f;
  float* __restrict__ wsz = a.ws + (size_t)units * npc * D * f + (size_t)u * npc * f;
  const float* __restrict__ S0 = nseg > 1 ? prefill_start_S(a, p, u, seg) : Sh;
  const float* __restrict__ z0 = nseg > 1 ? prefill_start_z(a, p, u, seg) : zh;

  // Starting state: zero for a delta, else the segment's, in the accumulator
  // layout.
  f32x16 sacc[C::NRT];
  if (delta) {
#pragma unroll
    for (int rt = 0; rt < C::NRT; ++rt) sacc[rt] = f32x16{};
    for (int r = tid; r < f; r += blockDim.x) sh.z[r] = 0.0f;
  } else {
#pragma unroll
    for (int rt = 0; rt < C::NRT; ++rt)
#pragma unroll
      for (int j = 0; j < 4; ++j) {  // rows rt*32 + j*8 + hh*4 .. +3: 16 bytes
        const f32x4 x = *reinterpret_cast<const f32x4*>(
            S0 + (size_t)col * f + rt * kTile + row_of(4 * j, hh));
#pragma unroll
        for (int r = 0; r < 4; ++r) sacc[rt][4 * j + r] = x[r];
      }
    for (int r = tid; r < f; r += blockDim.x) sh.z[r] = z0[r];
  }

  const T* __restrict__ Wt_h = (const T*)a.W + (size_t)h * F * D;
  op_t wop[FM::PPW][C::KD];  // W_h^T operands, kept for the whole prompt
  FM::load_w(Wt_h, w, li, hh, wop);
  const float scale = 1.0f / sqrtf((float)D);
  const float lw = want_out ? log_sigmoid(a.alpha[h]) : 0.0f;
  const bool row_ok = li < L;
  const int lrow = min(li, L - 1);

  // Block operands.  Unconditional, in-bounds loads: padding rows read row
  // L-1 and are zeroed by a select later; the prefetch past the segment's
  // last block re-reads that block.
  auto load_block = [&](int blk, op_t (&ko)[C::KD], op_t (&qo)[C::KD],
                        op_t (&vo)[C::KL]) {
    const size_t t0 = (size_t)blk * L;
    const T* kb = (const T*)a.k + (((size_t)b * T_ + t0) * Hkv + g) * D;
    const T* vb = (const T*)a.v + (((size_t)b * T_ + t0) * Hkv + g) * D;
    const T* krow = kb + (size_t)lrow * kstride + hh * E;
#pragma unroll
    for (int ks = 0; ks < C::KD; ++ks) ko[ks] = load_op<T>(krow + ks * KW);
#pragma unroll
    for (int ks = 0; ks < C::KL; ++ks)
      vo[ks] = load_rows_op<T>(vb + col, kstride, ks, hh, L, false);
    if (want_out) {
      const T* qrow = (const T*)a.q + (((size_t)b * T_ + t0) * Hq + h) * D +
                      (size_t)lrow * qstride + hh * E;
#pragma unroll
      for (int ks = 0; ks < C::KD; ++ks) qo[ks] = load_op<T>(qrow + ks * KW);
    }
  };
  op_t kop[C::KD], qop[C::KD], vop[C::KL];
#pragma unroll
  for (int ks = 0; ks < C::KD; ++ks) qop[ks] = M::zero();
  if (blk0 < blk1) load_block(blk0, kop, qop, vop);

  for (int blk = blk0; blk < blk1; ++blk) {
    const size_t t0 = (size_t)blk * L;
    op_t kn[C::KD], qn[C::KD], vn[C::KL];
#pragma unroll
    for (int ks = 0; ks < C::KD; ++ks) qn[ks] = M::zero();
    load_block(min(blk + 1, blk1 - 1), kn, qn, vn);
#pragma unroll
    for (int ks = 0; ks < C::KD; ++ks) {
      kop[ks] = keep_if<T>(row_ok, kop[ks]);
      qop[ks] = keep_if<T>(row_ok, qop[ks]);
    }

    lds_barrier();  // previous block's LDS readers are done
    float vk[FM::PPW][16], vq[FM::PPW][16];
    FM::logits(wop, kop, w, li, hh, vk, sh.fk);
    if (want_out) FM::logits(wop, qop, w, li, hh, vq, sh.fq);

    // In-block softmax branch (keys in rows, queries in columns).
    f32x16 acc_sm = {};
    float m = 0.0f, den = 1.0f;
    if (want_out) {
      f32x16 sc = {};
#pragma unroll
      for (int ks = 0; ks < C::KD; ++ks) sc = M::mma(kop[ks], qop[ks], sc);
      float p[16];
      m = -INFINITY;
#pragma unroll
      for (int i = 0; i < 16; ++i) {
        p[i] = row_of(i, hh) < L ? sc[i] * scale : -INFINITY;
        m = fmaxf(m, p[i]);
      }
      m = fmaxf(m, xor32(m));
      den = 0.0f;
#pragma unroll
      for (int i = 0; i < 16; ++i) {
        p[i] = row_of(i, hh) < L ? fast_exp(p[i] - m) : 0.0f;
        den += p[i];
      }
      den += xor32(den);
#pragma unroll
      for (int ks = 0; ks < C::KL; ++ks)
        acc_sm = mma_split_b<T>(vop[ks], &p[ks * E], acc_sm);
    }

    lds_barrier();
    FM::exps(w, li, hh, vk, sh.fk);
    if (want_out) FM::exps(w, li, hh, vq, sh.fq);
    lds_barrier();
    FM::normalise(w, li, hh, vk, sh.fk, [&](int f0, const float* x4) {
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const float x = row_ok ? x4[e] : 0.0f;
        const T hi = from_f32<T>(x);
        sh.phiKT[0][f0 + e][li] = hi;
        if constexpr (C::NPART == 2)
          sh.phiKT[1][f0 + e][li] = from_f32<T>(x - to_f32(hi));
      }
    });
    if (want_out) {
      // phi(q) to LDS and this wave's part of lin_den = phi(q) . z (the
      // features of the pairs it owns), summed over the waves below.
      float lz = 0.0f;
      FM::normalise(w, li, hh, vq, sh.fq, [&](int f0, const float* x4) {
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          sh.phiQ[li][f0 + e] = from_f32<T>(x4[e]);
          lz += x4[e] * sh.z[f0 + e];
        }
      });
      lz += xor32(lz);
      if (hh == 0) sh.lden[w][li] = lz;
    }
    lds_barrier();

    if (want_out) {
      // Readout against the state of the blocks before this one.
      f32x16 acc_lin = {};
      float lden = 0.0f;
#pragma unroll
      for (int ww = 0; ww < C::NW; ++ww) lden += sh.lden[ww][li];
#pragma unroll
      for (int ks = 0; ks < C::KF; ++ks) {
        const op_t pb = lds_op_perm<T>(&sh.phiQ[li][0], ks, hh, 0);
        op_t sa;
        if constexpr (E == 1) {
          sa = sacc[ks / 16][ks % 16];
        } else {
#pragma unroll
          for (int e = 0; e < E; ++e) {
            const int j = ks * E + e;  // flattened accumulator register
            sa[e] = (T)sacc[j / 16][j % 16];
          }
        }
        acc_lin = M::mma(sa, pb, acc_lin);
      }
      if (row_ok) {
        float ca = 1.0f, cz = 0.0f, rz = 0.0f;
        if (lden > 0.0f) {
          const float la = lw + m, lb = logf(lden);
          const float c = fmaxf(la, lb);
          ca = expf(la - c);
          cz = expf(lb - c);
          rz = 1.0f / lden;
        }
        const float inv = 1.0f / (ca * den + cz);
        const size_t obase = (((size_t)b * T_ + t0 + li) * Hq + h) * D;
#pragma unroll
        for (int i = 0; i < 16; i += 4) {
          float o[4];
#pragma unroll
          for (int e = 0; e < 4; ++e)
            o[e] = (ca * acc_sm[i + e] + cz * (acc_lin[i + e] * rz)) * inv;
          store_out4<T>(a.out, obase + w * kTile + row_of(i, hh), o, a.s.out_f32);
        }
      }
    }

    // Commit the block: S += phi(K)^T V in the accumulators.
#pragma unroll
    for (int rt = 0; rt < C::NRT; ++rt)
#pragma unroll
      for (int ks = 0; ks < C::KL; ++ks)
#pragma unroll
        for (int part = 0; part < C::NPART; ++part)
          sacc[rt] = M::mma(
              lds_op_perm<T>(&sh.phiKT[part][rt * kTile + li][0], ks, hh, 0),
              vop[ks], sacc[rt]);
    lds_barrier();  // every wave has read z for this block
    // z += sum_t phi(k_t): row r of phiKT holds the 32 tokens contiguously
    // (zero past the block length), read 16 bytes at a time.
    for (int r = tid; r < f; r += blockDim.x) {
      float s = 0.0f;
#pragma unroll
      for (int part = 0; part < C::NPART; ++part)
#pragma unroll
        for (int t0 = 0; t0 < kTile; t0 += 16 / (int)sizeof(T)) {
          const uint4 x = *reinterpret_cast<const uint4*>(&sh.phiKT[part][r][t0]);
          const T* xt = reinterpret_cast<const T*>(&x);
#pragma unroll
          for (int e = 0; e < 16 / (int)sizeof(T); ++e) s += to_f32(xt[e]);
        }
      sh.z[r] += s;
    }
#pragma unroll
    for (int ks = 0; ks < C::KD; ++ks) {
      kop[ks] = kn[ks];
      qop[ks] = qn[ks];
    }
#pragma unroll
    for (int ks = 0; ks < C::KL; ++ks) vop[ks] = vn[ks];
  }

  // A delta goes to the workspace; the last segment's walk writes the state.
  if (!delta && !last) return;
  float* dstS = delta ? wsS + (size_t)seg * D * f : Sh;
  float* dstz = delta ? wsz + (size_t)seg * f : zh;
#pragma unroll
  for (int rt = 0; rt < C::NRT; ++rt)
#pragma unroll
    for (int j = 0; j < 4; ++j)
      *reinterpret_cast<f32x4*>(dstS + (size_t)col * f + rt * kTile + row_of(4 * j, hh)) =
          f32x4{sacc[rt][4 * j], sacc[rt][4 * j + 1], sacc[rt][4 * j + 2], sacc[rt][4 * j + 3]};
  lds_barrier();
  for (int r = tid; r < f; r += blockDim.x) dstz[r] = sh.z[r];
}


// ---------------------------------------------------------------------------
// Pipelined walk (bf16, F <= 64, outputs wanted): one workgroup per (request,
// head, segment), 4 + D/32 waves.  The roles work on different blocks of the
// segment and meet at one barrier per iteration; in iteration it:
//   QS waves (0, 1: even and odd blocks): phi(Q) and the in-block softmax of
//     a block over two iterations -- the logits, the scores, the first
//     exponentials and the softmax rows of block it+1, then the rest of
//     phi(Q) of block it, its store and the store of P (a bf16 pair hi + lo);
//     with the second half, z_it = z_{it-1} + phi(K_{it-1})^T 1 (MFMAs);
//   K waves (2, 3): phi(K) likewise, stored as rows of hi and lo planes
//     (TokTile); with the first half of block it+1, the output store of block
//     it-3 (whole rows, from the staging tile the state waves filled an
//     iteration before), then lin_den = phi(Q) z of block it-1 (on the MFMAs, z
//     as three bf16 parts, which hold all of its bits) and its merge
//     coefficients;
//   state waves (D/32): the merge of block it-2 (two coefficients per row)
//     into staging; then, for block it-1: the V^T operands of the wave's 32 columns, the readout
//     phi(Q) S against the state of the blocks before it, P V of its
//     columns and the commit into S columns 32w .. 32w+31 (fp32
//     accumulators).
// The QS and K waves hand a block to the state waves through a double
// buffer (written in iteration c, read in c+1), the merge coefficients
// through a second (written in c+1, read in c+2); z goes from one QS wave to
// the other through a triple buffer (z_c is written in iteration c and read
// in c+1).
// Operand precision is that of the single-group walk above, except that lin_den
// takes phi(Q) as the readout does, in bf16; the merge's exponentials, logarithm
// and reciprocals are the hardware's, about 1 ulp each.
// A block step is bound by the longest role between two barriers, and by what
// two waves of a SIMD issue together, so the hand-over costs no instructions
// that only move bits: phi(K)^T and V^T operands come from row-major tiles by
// transposing LDS reads (as hi | lo pairs in dwords they took 72 byte permutes
// per state wave and block, V^T 16 masked two-byte reads, and lin_den 130 VALU
// instructions); and the state waves, the longest role, load nothing behind a
// store (their wait for V's rows had counted the block's output store, issued
// just before: 1,700 of 5,000 cycles a block).  8 x 8192 tokens: 385 us before,
// 355 us with the increments below changed alike.
// ---------------------------------------------------------------------------
template <typename T, int D, int F>
struct PrefillPipeCfg {
  typedef Mma<T> M;
  typedef typename M::op_t op_t;
  static constexpr int NC = D / kTile;  // state waves
  static constexpr int NWAVE = 4 + NC;
  static constexpr int f = 2 * F;
  static constexpr int NT = F / kTile;
  static constexpr int NPAIR = 2 * NT;
  static constexpr int NRT = f / kTile;
  static constexpr int KD = D / M::KW;
  static constexpr int KL = kTile / M::KW;
  static constexpr int KF = f / M::KW;
  // Row strides of the bf16 tiles read as 8-byte pieces by 32 lanes at a
  // time: an odd number of dword pairs, so that the 32 rows fall in distinct
  // bank pairs.
  static constexpr int QLD = f + 4, PLD = kTile + 4;
  struct alignas(16) Buf {            // written in iteration c, read in c + 1
    T phiQ[kTile][QLD];               // phi(q_i)[r] at [i][r]
    T phiK[2][kTile * f];             // phi(k_t): planes hi and lo (TokTile)
    T ph[kTile][PLD];                 // P (relative to the row max) as hi + lo,
    T pl[kTile][PLD];                 //   [query][key]
    float m[kTile], den[kTile];       // row max and sum of the block scores
  };
  struct alignas(16) Smem {
    Buf buf[2];
    float2 coef[2][kTile];            // merge: out = x P V + y phi(Q) S per row
    float z[3][f];                    // z_c at [(c - first block) % 3]
    T zp[3][3][f];                    // and as three parts, their sum exactly z_c
    float stage[2][kTile][D + 4];     // merged outputs of a block, [row][column]; as
                                      // bf16, rows of 2D bytes (StageRow)
    T vt[NC][kTile][kTile];           // V rows of each state wave's columns
  };
};

// Byte offset of columns c .. c+3 of row t of a staged bf16 tile: 16-byte
// chunk c/8 at (c/8) ^ (t % 16) (D = 128; ^ (t / 2 % 8) for D = 64), its 8-byte
// halves swapped in rows 16 .. 31, so that the same columns of 32 rows (a
// write) fall in distinct banks, as whole rows (a read) do.
template <int D>
struct StageRow {
  __device__ static inline int swz(int t) { return D == 128 ? t & 15 : (t >> 1) & 7; }
  __device__ static inline int at(int t, int c) {
    return t * D * 2 + (((c >> 3) ^ swz(t)) * 16) + ((((c >> 2) ^ (t >> 4)) & 1) * 8);
  }
};

// Four floats as three bf16 parts each: x = p0 + p1 + p2 (8 significant bits
// apiece cover the 24 of x).
__device__ inline void split_three4(const f32x4& x, bf16x4& p0, bf16x4& p1, bf16x4& p2) {
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    p0[e] = (bf16)x[e];
    const float r = x[e] - (float)p0[e];
    p1[e] = (bf16)r;
    p2[e] = (bf16)(r - (float)p1[e]);
  }
}

template <int D>
constexpr int pipe_threads() {
  return kWave * (4 + D / kTile);
}

template <typename T, int D, int F>
__global__ __launch_bounds__(pipe_threads<D>()) void hyb_prefill_pipe_kernel(
    PrefillArgs a, SegPlan p) {
  typedef PrefillPipeCfg<T, D, F> C;
  typedef typename C::M M;
  typedef typename C::op_t op_t;
  typedef WaveFeatMap<T, D, F> WFM;
  typedef TokTile<2 * F> Tok;
  constexpr int f = C::f, E = M::E, KW = M::KW, NT = C::NT, NC = C::NC;
  static_assert(sizeof(T) == 2, "the pipelined walk is the bf16 path");
  static_assert(pipe_threads<D>() == kWave * C::NWAVE, "launch bounds match the waves");
  __shared__ typename C::Smem sh;

  // The wave index through readfirstlane: the compiler then knows it is
  // uniform, and the role branches below are scalar jumps, not exec masks.
  const int tid = threadIdx.x, lane = tid & (kWave - 1);
  const int w = __builtin_amdgcn_readfirstlane(tid / kWave);
  const int li = lane & 31, hh = lane >> 5;
  const int Hq = a.s.Hq, Hkv = a.s.Hkv, L = a.s.L, T_ = a.T;
  const int units = a.s.B * Hq, nseg = p.nseg;
  const int vix = xcd_unit(blockIdx.x, units * nseg);
  const int u = vix % units, seg = vix / units;
  const int b = u / Hq, h = u % Hq, g = h / (Hq / Hkv);
  const int slot = a.slots ? a.slots[b] : b;
  const bool last = seg == nseg - 1;
  const size_t qstride = (size_t)Hq * D, kstride = (size_t)Hkv * D;
  const int nblk = T_ / L;
  const int blk0 = seg * p.sb, blk1 = min(nblk, blk0 + p.sb);
  const int nit = blk1 - blk0 + 4;  // iterations blk0-1 .. blk1+2
  if (slot < 0 || slot >= a.s.n_slots) {  // uniform per workgroup
    const size_t ob = ((size_t)b * T_ * Hq + h) * D;
    for (int t = blk0 * L; t < blk1 * L; ++t)
      for (int c = tid; c < D; c += blockDim.x)
        store_out1<T>(a.out, ob + (size_t)t * qstride + c, __builtin_nanf(""), a.s.out_f32);
    return;
  }
  const bool row_ok = li < L;
  const int lrow = min(li, L - 1);
  // Raw buffers over this request's rows of q, k and v: a block's offset is
  // a scalar, a lane's row offset one 32-bit register, a k-step's the
  // immediate (the launcher keeps a request's rows under 2 GiB).
  const __amdgpu_buffer_rsrc_t qrs = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<T*>((const T*)a.q + (size_t)b * T_ * qstride), 0, (int)(T_ * qstride * sizeof(T)),
      kBufferWord3);
  const __amdgpu_buffer_rsrc_t krs = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<T*>((const T*)a.k + (size_t)b * T_ * kstride), 0, (int)(T_ * kstride * sizeof(T)),
      kBufferWord3);
  const __amdgpu_buffer_rsrc_t vrs = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<T*>((const T*)a.v + (size_t)b * T_ * kstride), 0, (int)(T_ * kstride * sizeof(T)),
      kBufferWord3);
  const int qlane = (lrow * (int)qstride + hh * E) * (int)sizeof(T);
  const int klane = (lrow * (int)kstride + hh * E) * (int)sizeof(T);
  auto qoff = [&](int blk) { return (int)(((size_t)blk * L * qstride + (size_t)h * D) * sizeof(T)); };
  auto koff = [&](int blk) { return (int)(((size_t)blk * L * kstride + (size_t)g * D) * sizeof(T)); };
  // Rows of a block tile as operands (rows past the block length read row
  // L-1; the roles mask them).
  auto load_q = [&](int blk, op_t (&o)[C::KD]) {
    const int so = qoff(blk);
#pragma unroll
    for (int ks = 0; ks < C::KD; ++ks) o[ks] = buf_op<T>(qrs, qlane + ks * KW * (int)sizeof(T), so);
  };
  auto load_k = [&](int blk, op_t (&o)[C::KD]) {
    const int so = koff(blk);
#pragma unroll
    for (int ks = 0; ks < C::KD; ++ks) o[ks] = buf_op<T>(krs, klane + ks * KW * (int)sizeof(T), so);
  };

  // Set-up: the segment's starting z into z[0].
  {
    const float* __restrict__ z0 = nseg > 1 ? prefill_start_z(a, p, u, seg) : a.z + ((size_t)slot * Hq + h) * f;
    for (int r = 4 * tid; r < f; r += 4 * C::NWAVE * kWave) {
      const f32x4 x = *reinterpret_cast<const f32x4*>(z0 + r);
      *reinterpret_cast<f32x4*>(&sh.z[0][r]) = x;
      split_three4(x, *reinterpret_cast<bf16x4*>(&sh.zp[0][0][r]), *reinterpret_cast<bf16x4*>(&sh.zp[0][1][r]),
                   *reinterpret_cast<bf16x4*>(&sh.zp[0][2][r]));
    }
  }
  lds_barrier();  // z ready

  constexpr float kLog2e = 1.4426950408889634f;
  // logits U^T = W^T X^T of the rows x (W_h^T is held in the feature-map waves'
  // registers, wop)
  auto logits = [&](const op_t (&wop)[NT][C::KD], const op_t (&x)[C::KD], float (&phi)[C::NPAIR][16]) {
#pragma unroll
    for (int t = 0; t < NT; ++t) {
      f32x16 acc = {};
#pragma unroll
      for (int ks = 0; ks < C::KD; ++ks) acc = M::mma(wop[t][ks], x[ks], acc);
#pragma unroll
      for (int i = 0; i < 16; ++i) phi[t][i] = acc[i];
    }
  };
  // Feature-map halves: the row extremes, every first-sign exponential and
  // the first NA of the second sign (the other second-sign slots keep the
  // logit); then the rest, the sums and the normalisation (keep = row_ok
  // zeroes a padding row).  e^(u - mx) = 2^(u log2 e - mx log2 e): one fma
  // per exponent; the rounding of mx log2 e is common to the row and cancels
  // in the ratio.
  auto fm_first = [&](float (&phi)[C::NPAIR][16], int NA, float& mnl, float& sp, float& sn) {
    float mx = -INFINITY, mn = INFINITY;
#pragma unroll
    for (int t = 0; t < NT; ++t)
#pragma unroll
      for (int i = 0; i < 16; ++i) {
        mx = fmaxf(mx, phi[t][i]);
        mn = fminf(mn, phi[t][i]);
      }
    mx = fmaxf(mx, xor32(mx));
    mn = fminf(mn, xor32(mn));
    const float mxl = mx * kLog2e;
    mnl = mn * kLog2e;
    sp = 0.0f;
    sn = 0.0f;
#pragma unroll
    for (int t = 0; t < NT; ++t)
#pragma unroll
      for (int i = 0; i < 16; ++i) {
        const float uu = phi[t][i];
        if (t * 16 + i < NA) {
          phi[NT + t][i] = __builtin_amdgcn_exp2f(__builtin_fmaf(-uu, kLog2e, mnl));
          sn += phi[NT + t][i];
        } else {
          phi[NT + t][i] = uu;
        }
        phi[t][i] = __builtin_amdgcn_exp2f(__builtin_fmaf(uu, kLog2e, -mxl));
        sp += phi[t][i];
      }
  };
  auto fm_second = [&](float (&phi)[C::NPAIR][16], int NA, float mnl, float sp, float sn) {
#pragma unroll
    for (int t = 0; t < NT; ++t)
#pragma unroll
      for (int i = 0; i < 16; ++i) {
        if (t * 16 + i < NA) continue;
        phi[NT + t][i] = __builtin_amdgcn_exp2f(__builtin_fmaf(-phi[NT + t][i], kLog2e, mnl));
        sn += phi[NT + t][i];
      }
    sp += xor32(sp);
    sn += xor32(sn);
    const float ip = row_ok ? 1.0f / sp : 0.0f, in = row_ok ? 1.0f / sn : 0.0f;
#pragma unroll
    for (int t = 0; t < NT; ++t)
#pragma unroll
      for (int i = 0; i < 16; ++i) {
        phi[t][i] *= ip;
        phi[NT + t][i] *= in;
      }
  };

  if (w < 4) {
    // ---- QS waves (0, 1) and K waves (2, 3): blocks c = blk0 + par + 2j;
    // the first half of block c in iteration c-1, the second in iteration c;
    // the odd wave idles in the first iteration, and both idle after their
    // last block, so that every wave passes nit barriers, as the state waves
    // do ----
    const int par = w & 1;
    op_t ones;
#pragma unroll
    for (int e = 0; e < E; ++e) ones[e] = (T)1.0f;
    auto role = [&](auto key) {
      constexpr bool K = decltype(key)::value;
      // phi(K) stores more (the hi | lo pairs), so it moves more of its
      // exponentials into the first half
      constexpr int NA = K ? NT * 8 : 0;
      op_t x[C::KD], xk[K ? 1 : C::KD], wop[NT][C::KD];
      WFM::load_w((const T*)a.W + (size_t)h * F * D, li, hh, wop);
      auto load = [&](int blk) {
        if constexpr (K) {
          load_k(blk, x);
        } else {
          load_q(blk, x);
          load_k(blk, xk);
        }
      };
      if (blk0 + par < blk1) load(blk0 + par);
      int nbar = 0;
      if (par) {
        lds_barrier();
        ++nbar;
      }
      const float scale = 1.0f / sqrtf((float)D);
      const float lw = log_sigmoid(a.alpha[h]);
      // K: the output store of block c, whole rows (D/8 lanes per row, 8
      // columns each), a scalar base and 32-bit lane offsets
      const bool out_f32 = a.s.out_f32;
      auto store_rows = [&](int c) __attribute__((always_inline)) {
        constexpr int LPR = D / 8, RPP = kWave / LPR, NP = kTile / RPP;  // lanes per row, rows per pass
        const char* st = reinterpret_cast<const char*>(sh.stage[(c - blk0) & 1]);
        int l = lane;  // (opaque: addresses are formed here, not kept across the loop)
        asm volatile("" : "+v"(l));
        const int r0 = l / LPR, c8 = l % LPR * 8;
        const size_t row = (size_t)b * T_ + (size_t)c * L;
        if (out_f32) {
          char* ob = (char*)a.out + (row * qstride + (size_t)h * D) * 4;
#pragma unroll 2
          for (int p = 0; p < NP; ++p) {
            const int t = p * RPP + r0;
            const f32x4* s = reinterpret_cast<const f32x4*>(&sh.stage[(c - blk0) & 1][t][c8]);
            const f32x4 x0 = s[0], x1 = s[1];
            if (t < L) {
              f32x4* o = reinterpret_cast<f32x4*>(ob + (unsigned)((t * (int)qstride + c8) * 4));
              o[0] = x0;
              o[1] = x1;
            }
          }
        } else {
          char* ob = (char*)a.out + (row * qstride + (size_t)h * D) * sizeof(T);
          u32x4 x[NP];
#pragma unroll
          for (int p = 0; p < NP; ++p) x[p] = *reinterpret_cast<const u32x4*>(st + (StageRow<D>::at(p * RPP + r0, c8) & ~15));
          __builtin_amdgcn_sched_barrier(0);
#pragma unroll
          for (int p = 0; p < NP; ++p) {
            const int t = p * RPP + r0;
            if (p * RPP >= 16) x[p] = u32x4{x[p][2], x[p][3], x[p][0], x[p][1]};
            if (t < L) *reinterpret_cast<u32x4*>(ob + (unsigned)((t * (int)qstride + c8) * 2)) = x[p];
          }
        }
      };
      // QS: z_{c+1} = z_c + phi(K_c)^T 1 from the tile of block c, as
      // accumulator tiles of 16 features whose columns are all equal: lane
      // column ft keeps tile ft, so one lane row holds all of z.
      auto z_update = [&](int c) __attribute__((always_inline)) {
        const typename C::Buf& Bc = sh.buf[(c - blk0) & 1];
        int l = lane;  // (opaque, as above)
        asm volatile("" : "+v"(l));
        const int zb = Tok::sum_base(l), ft = l & 15;
        const int r = (min(ft, f / 16 - 1)) * 16 + (l >> 4) * 4;
        const f32x4 zc = *reinterpret_cast<const f32x4*>(&sh.z[(c - blk0) % 3][r]);
        f32x4 sum = {};
#pragma unroll
        for (int f0 = 0; f0 < f / 16; f0 += 4) {
          op_t kh[4], kl[4];
#pragma unroll
          for (int j = 0; j < 4; ++j) {
            kh[j] = Tok::sum_op(Bc.phiK[0], zb, f0 + j);
            kl[j] = Tok::sum_op(Bc.phiK[1], zb, f0 + j);
          }
          __builtin_amdgcn_sched_barrier(0);
          f32x4 dz[4];
#pragma unroll
          for (int j = 0; j < 4; ++j) dz[j] = Mma16<T>::mma(kh[j], ones, f32x4{});
#pragma unroll
          for (int j = 0; j < 4; ++j) dz[j] = Mma16<T>::mma(kl[j], ones, dz[j]);
#pragma unroll
          for (int j = 0; j < 4; ++j)
#pragma unroll
            for (int e = 0; e < 4; ++e) sum[e] = ft == f0 + j ? dz[j][e] : sum[e];
        }
        const f32x4 zn = zc + sum;
        bf16x4 p0, p1, p2;
        split_three4(zn, p0, p1, p2);
        if (ft < f / 16) {
          const int n = (c + 1 - blk0) % 3;
          *reinterpret_cast<f32x4*>(&sh.z[n][r]) = zn;
          *reinterpret_cast<bf16x4*>(&sh.zp[n][0][r]) = p0;
          *reinterpret_cast<bf16x4*>(&sh.zp[n][1][r]) = p1;
          *reinterpret_cast<bf16x4*>(&sh.zp[n][2][r]) = p2;
          if (last && c + 1 == blk1) *reinterpret_cast<f32x4*>(a.z + ((size_t)slot * Hq + h) * f + r) = zn;
        }
      };
      // lin_den = phi(q) . z of block c and the two merge coefficients of
      // each row, for the state waves' merge of block c an iteration later:
      // out = (ca P V + cz phi(Q) S / lin_den) / (ca den + cz), with the
      // overflow-safe ca, cz of the single-group walk; lin_den <= 0 leaves
      // the in-block softmax alone.
      auto coefs = [&](int c) {
        const typename C::Buf& Bc = sh.buf[(c - blk0) & 1];
        // rows 0, 1, 2 of the left operand: the parts of z (the other rows
        // repeat the last and are not read); columns: the queries
        const T* zr = sh.zp[(c - blk0) % 3][min(li, 2)];
        f32x16 ld = {};
#pragma unroll
        for (int k0 = 0; k0 < C::KF; k0 += 4) {
          op_t za[4], qa[4];
#pragma unroll
          for (int j = 0; j < 4; ++j) {
            za[j] = lds_op_perm<T>(zr, k0 + j, hh, 0);
            qa[j] = lds_op_perm<T>(&Bc.phiQ[li][0], k0 + j, hh, 0);
          }
          __builtin_amdgcn_sched_barrier(0);
#pragma unroll
          for (int j = 0; j < 4; ++j) ld = M::mma(za[j], qa[j], ld);
        }
        const float lden = ld[0] + (ld[1] + ld[2]);  // (lanes of the lower half)
        const float m = Bc.m[li], den = Bc.den[li];
        float ca = 1.0f, cz = 0.0f, rz = 0.0f;
        if (lden > 0.0f) {
          // (the hardware's logarithm and reciprocal take a subnormal as zero)
          const float up = lden < 0x1p-100f ? 0x1p64f : 1.0f, x = lden * up;
          const float la = (lw + m) * kLog2e, lb = __builtin_amdgcn_logf(x) - (up > 1.0f ? 64.0f : 0.0f);
          const float cc = fmaxf(la, lb);
          ca = __builtin_amdgcn_exp2f(la - cc);
          cz = __builtin_amdgcn_exp2f(lb - cc);
          rz = fast_rcp(x) * up;
        }
        const float inv = fast_rcp(ca * den + cz);
        if (hh == 0) sh.coef[(c - blk0) & 1][li] = make_float2(ca * inv, cz * rz * inv);
      };
      for (int c = blk0 + par; c < blk1; c += 2) {
        // ---- iteration c-1 ----
        if constexpr (K) {
          if (c - 4 >= blk0) store_rows(c - 4);
          if (c - 2 >= blk0) coefs(c - 2);
        }
        float phi[C::NPAIR][16];
        logits(wop, x, phi);
        f32x16 sc = {};
        if constexpr (!K) {
          // scores: keys in rows, queries in columns
#pragma unroll
          for (int ks = 0; ks < C::KD; ++ks)
            sc = M::mma(xk[ks], x[ks], sc);  // (rows past L repeat row L-1: masked below, or not stored)
        }
        // (the operands are read by the products above before the rows of
        // this wave's next block land in the same registers)
        __builtin_amdgcn_sched_barrier(0);
        if (c + 2 < blk1) load(c + 2);
        float mnl, sp, sn;
        fm_first(phi, NA, mnl, sp, sn);
        float pr[16], m = 0.0f, den = 0.0f;
        if constexpr (!K) {
          m = -INFINITY;
#pragma unroll
          for (int i = 0; i < 16; ++i) {
            pr[i] = row_of(i, hh) < L ? sc[i] * scale : -INFINITY;
            m = fmaxf(m, pr[i]);
          }
          m = fmaxf(m, xor32(m));
#pragma unroll
          for (int i = 0; i < 16; ++i) {
            pr[i] = row_of(i, hh) < L ? fast_exp(pr[i] - m) : 0.0f;
            den += pr[i];
          }
          den += xor32(den);
        }
        lds_barrier();
        // ---- iteration c ----
        if constexpr (!K) {
          if (c - 1 >= blk0) z_update(c - 1);
        }
        fm_second(phi, NA, mnl, sp, sn);
        typename C::Buf& B = sh.buf[(c - blk0) & 1];
        if constexpr (!K) {
#pragma unroll
          for (int p = 0; p < C::NPAIR; ++p)
#pragma unroll
            for (int i = 0; i < 16; ++i) B.phiQ[li][WFM::feature(16 * p + i, hh)] = from_f32<T>(phi[p][i]);
          // P of query li, keys row_of(i, hh): runs of 4 consecutive keys
#pragma unroll
          for (int i = 0; i < 16; i += 4) {
            bf16x4 hi4, lo4;
            split_hi_lo4(&pr[i], hi4, lo4);
            *reinterpret_cast<bf16x4*>(&B.ph[li][row_of(i, hh)]) = hi4;
            *reinterpret_cast<bf16x4*>(&B.pl[li][row_of(i, hh)]) = lo4;
          }
          if (hh == 0) {
            B.m[li] = m;
            B.den[li] = den;
          }
        } else {
          char* kt = reinterpret_cast<char*>(B.phiK[0]);
          // (opaque: the piece addresses are formed here, not kept in registers
          // across the loop, where they would spill)
          int wb = Tok::write_base(li, hh);
          asm volatile("" : "+v"(wb));
#pragma unroll
          for (int p = 0; p < C::NPAIR; ++p)
#pragma unroll
            for (int i = 0; i < 16; i += 4) {  // features 32p + 2i + 4hh ..
              bf16x4 hi4, lo4;
              split_hi_lo4(&phi[p][i], hi4, lo4);
              const int at = wb ^ (16 * (4 * p + i / 4));
              *reinterpret_cast<bf16x4*>(kt + at) = hi4;
              *reinterpret_cast<bf16x4*>(kt + at + Tok::kPlane * 2) = lo4;
            }
        }
        lds_barrier();
        nbar += 2;
      }
      // what is left of the earlier blocks, each in its iteration: the output
      // stores and the last coefficients (K), the last z (QS)
      int c = blk0 + par;
      if (c < blk1) c += (blk1 - c + 1) / 2 * 2;
      for (; c - 1 <= blk1 + 2; c += 2) {
        if constexpr (K) {
          if (c - 4 >= blk0 && c - 4 < blk1) store_rows(c - 4);
          if (c - 2 >= blk0 && c - 2 < blk1) coefs(c - 2);
        }
        lds_barrier();
        ++nbar;
        if (c > blk1 + 2) break;
        if constexpr (!K) {
          if (c - 1 >= blk0 && c - 1 < blk1) z_update(c - 1);
        }
        lds_barrier();
        ++nbar;
      }
      for (; nbar < nit; ++nbar) lds_barrier();
    };
    if (w >= 2) role(std::true_type{});
    else role(std::false_type{});
  } else {
    // ---- state waves: merge and store of block it-2; V^T, readout, P V
    // and commit of block it-1 ----
    const int cw = w - 4;
    const int col = cw * kTile + li;
    const size_t sbase = (size_t)slot * Hq + h;
    float* __restrict__ Sh = a.S + sbase * f * D;
    const float* __restrict__ S0 = nseg > 1 ? prefill_start_S(a, p, u, seg) : Sh;
    // S columns col of all f rows, the segment's starting state.
    // (Declared here, not before the role branches: a value live across the
    // other roles' code takes registers there too.)
    f32x16 sacc[C::NRT];
#pragma unroll
    for (int rt = 0; rt < C::NRT; ++rt)
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const f32x4 x = *reinterpret_cast<const f32x4*>(S0 + (size_t)col * f + rt * kTile + row_of(4 * j, hh));
#pragma unroll
        for (int r = 0; r < 4; ++r) sacc[rt][4 * j + r] = x[r];
      }
    // V rows of this wave's 32 columns, one block ahead: 4 lanes per row
    // (16 bytes each), 16 rows per load; a row at or past the block length
    // reads past the buffer's end, as zeros.  The V^T operands (lane li:
    // column 32cw + li; k-step ks: the tokens row_of(ks*E + e, hh), the order
    // in which P and phi(K)^T enter the products) are then read, transposed,
    // from this wave's LDS copy of the rows (four rows are all of the banks).
    int vlane[2];
#pragma unroll
    for (int s2 = 0; s2 < 2; ++s2) {
      const int t = s2 * 16 + (lane >> 2);
      vlane[s2] = t < L ? (t * (int)kstride + cw * kTile + (lane & 3) * 8) * (int)sizeof(T) : kPastBuffer;
    }
    op_t vrow[2];
    auto load_v = [&](int blk) {
      const int so = koff(blk);
#pragma unroll
      for (int s2 = 0; s2 < 2; ++s2) vrow[s2] = buf_op<T>(vrs, vlane[s2], so);
    };
    T (*vt)[kTile] = sh.vt[cw];
    const int krb0 = Tok::read_base(lane);
    const T* vtr = &vt[4 * hh + ((lane & 15) >> 2)][16 * ((lane >> 4) & 1) + 4 * (lane & 3)];
    if (blk0 < blk1) load_v(blk0);
    // the products of a block, kept from its iteration to its merge in the
    // next
    f32x16 olin = {}, apv = {};
    constexpr int RH = (C::NRT + 1) / 2;
    // The merge of block cm into the staging tile (this wave's columns),
    // which the K waves store after the next barrier.
    const bool out_f32 = a.s.out_f32;
    auto merge = [&](int cm, const float2& cf) __attribute__((always_inline)) {
      float (*st)[D + 4] = sh.stage[(cm - blk0) & 1];
      if (out_f32) {
#pragma unroll
        for (int i = 0; i < 16; i += 4) {
          f32x4 o;
#pragma unroll
          for (int e = 0; e < 4; ++e) o[e] = cf.x * apv[i + e] + cf.y * olin[i + e];
          *reinterpret_cast<f32x4*>(&st[li][cw * kTile + row_of(i, hh)]) = o;
        }
      } else {
        char* sb = reinterpret_cast<char*>(st);
#pragma unroll
        for (int i = 0; i < 16; i += 4) {
          bf16x4 o;
#pragma unroll
          for (int e = 0; e < 4; ++e) o[e] = (T)(cf.x * apv[i + e] + cf.y * olin[i + e]);
          *reinterpret_cast<bf16x4*>(sb + StageRow<D>::at(li, cw * kTile + row_of(i, hh))) = o;
        }
      }
    };
    lds_barrier();  // iterations blk0-1 and blk0: nothing to do yet
    lds_barrier();
    for (int cr = blk0; cr < blk1; ++cr) {  // iteration cr + 1
      const int cm = cr - 1;
      {
        typename C::Buf& B = sh.buf[(cr - blk0) & 1];
        int krb = krb0;  // (opaque: the operand addresses are formed per block)
        asm volatile("" : "+v"(krb));
        // V rows of block cr through this wave's LDS tile (its own writes
        // complete before its reads), the next block's rows issued
#pragma unroll
        for (int s2 = 0; s2 < 2; ++s2)
          *reinterpret_cast<op_t*>(&vt[s2 * 16 + (lane >> 2)][(lane & 3) * 8]) = vrow[s2];
        __builtin_amdgcn_sched_barrier(0);
        if (cr + 1 < blk1) load_v(cr + 1);
        // LDS operands are requested in batches ahead of the products that
        // use them, a scheduling barrier after each batch: fetched one at a
        // time next to its product, every operand costs a full LDS round
        // trip.  Batch 1: the coefficients of the block before, the
        // operands of the readout and V^T.
        const float2 cf = sh.coef[(cm - blk0) & 1][li];
        asm volatile("" ::: "memory");
        op_t pb[C::KF];
#pragma unroll
        for (int ks = 0; ks < C::KF; ++ks) pb[ks] = lds_op_perm<T>(&B.phiQ[li][0], ks, hh, 0);
        op_t vk[C::KL];
#pragma unroll
        for (int ks = 0; ks < C::KL; ++ks)
          vk[ks] = lds_tr_op(vtr + 16 * ks * kTile, vtr + (16 * ks + 8) * kTile);
        __builtin_amdgcn_sched_barrier(0);
        if (cm >= blk0) merge(cm, cf);
        __builtin_amdgcn_sched_barrier(0);
        // readout against the state of the blocks before cr
        f32x16 ol = {};
#pragma unroll
        for (int ks = 0; ks < C::KF; ++ks) {
          op_t sa;
#pragma unroll
          for (int e = 0; e < E; ++e) {
            const int j = ks * E + e;
            sa[e] = (T)sacc[j / 16][j % 16];
          }
          ol = M::mma(sa, pb[ks], ol);
        }
        __builtin_amdgcn_sched_barrier(0);
        // Batch 2: P of block cr and the commit operands of the first half
        // of the row tiles.
        op_t pph[C::KL], ppl[C::KL];
        op_t kh[RH][C::KL], kl[RH][C::KL];
#pragma unroll
        for (int ks = 0; ks < C::KL; ++ks) {
          pph[ks] = lds_op_perm<T>(&B.ph[li][0], ks, hh, 0);
          ppl[ks] = lds_op_perm<T>(&B.pl[li][0], ks, hh, 0);
        }
#pragma unroll
        for (int rt = 0; rt < RH; ++rt)
#pragma unroll
          for (int ks = 0; ks < C::KL; ++ks) {
            kh[rt][ks] = Tok::op(B.phiK[0], krb, rt, ks);
            kl[rt][ks] = Tok::op(B.phiK[1], krb, rt, ks);
          }
        __builtin_amdgcn_sched_barrier(0);
        // P V of this wave's columns (P as a bf16 pair hi + lo)
        f32x16 pv = {};
#pragma unroll
        for (int ks = 0; ks < C::KL; ++ks) {
          pv = M::mma(vk[ks], pph[ks], pv);
          pv = M::mma(vk[ks], ppl[ks], pv);
        }
        // commit: S += phi(K)^T V (this wave's columns), first half
#pragma unroll
        for (int rt = 0; rt < RH; ++rt)
#pragma unroll
          for (int ks = 0; ks < C::KL; ++ks) {
            sacc[rt] = M::mma(kh[rt][ks], vk[ks], sacc[rt]);
            sacc[rt] = M::mma(kl[rt][ks], vk[ks], sacc[rt]);
          }
        __builtin_amdgcn_sched_barrier(0);
        // Batch 3: the commit operands of the other row tiles.
        op_t kh2[C::NRT - RH][C::KL], kl2[C::NRT - RH][C::KL];
#pragma unroll
        for (int rt = RH; rt < C::NRT; ++rt)
#pragma unroll
          for (int ks = 0; ks < C::KL; ++ks) {
            kh2[rt - RH][ks] = Tok::op(B.phiK[0], krb, rt, ks);
            kl2[rt - RH][ks] = Tok::op(B.phiK[1], krb, rt, ks);
          }
        __builtin_amdgcn_sched_barrier(0);
        // commit, second half
#pragma unroll
        for (int rt = RH; rt < C::NRT; ++rt)
#pragma unroll
          for (int ks = 0; ks < C::KL; ++ks) {
            sacc[rt] = M::mma(kh2[rt - RH][ks], vk[ks], sacc[rt]);
            sacc[rt] = M::mma(kl2[rt - RH][ks], vk[ks], sacc[rt]);
          }
        olin = ol;
        apv = pv;
      }
      lds_barrier();
    }
    // iterations blk1+1 and blk1+2: the last block's merge (and its store)
    merge(blk1 - 1, sh.coef[(blk1 - 1 - blk0) & 1][li]);
    lds_barrier();
    lds_barrier();
    if (last) {
#pragma unroll
      for (int rt = 0; rt < C::NRT; ++rt)
#pragma unroll
        for (int j = 0; j < 4; ++j)
          *reinterpret_cast<f32x4*>(Sh + (size_t)col * f + rt * kTile + row_of(4 * j, hh)) =
              f32x4{sacc[rt][4 * j], sacc[rt][4 * j + 1], sacc[rt][4 * j + 2], sacc[rt][4 * j + 3]};
    }
  }
}


// ---------------------------------------------------------------------------
// Pipelined increment (bf16, F <= 64): the increment of one piece of the
// plan, dS = sum_c phi(K_c)^T V_c and dz = sum_c sum_t phi(k_t), a pair of
// blocks per iteration, 4 + D/32 waves:
//   feature-map waves (4): phi(K) of the piece's blocks, wave w taking the
//     blocks 4m + w; a map spans two iterations (the logits, the row extremes
//     and most exponentials, then the rest and the store of phi(K) as rows of
//     hi and lo planes, TokTile), so the four waves finish a pair per
//     iteration;
//   state waves (D/32): the commit of the previous pair into S columns
//     32w .. 32w+31 and dz (as phi(K)^T 1) in fp32 accumulators, with the V^T
//     operands of their columns from whole V rows through a per-wave LDS
//     tile.
// One barrier per iteration; phi(K) is double-buffered (written in iteration
// j for pair j, read in j + 1).  Bound by the state waves' LDS reads (44 KB a
// wave and pair) between their products; 8 x 8192 tokens without outputs: 138 us
// with phi(K)^T as hi | lo pairs in dwords and V^T by an identity product,
// 115 us with transposing reads.  Requesting each batch of operands a batch
// ahead of its products was slower (122 us).
// ---------------------------------------------------------------------------
template <typename T, int D, int F>
struct DeltaPipeCfg {
  typedef Mma<T> M;
  typedef typename M::op_t op_t;
  static constexpr int NC = D / kTile;   // state waves
  static constexpr int NWAVE = 4 + NC;
  static constexpr int f = 2 * F;
  static constexpr int NT = F / kTile;
  static constexpr int NPAIR = 2 * NT;
  static constexpr int NRT = f / kTile;
  static constexpr int ZPW = (NRT + NC - 1) / NC;  // z tiles per state wave
  static constexpr int KD = D / M::KW;
  static constexpr int KL = kTile / M::KW;
  typedef WaveFeatMap<T, D, F> WFM;
  struct alignas(16) Buf {
    T phiK[2][2][kTile * f];             // per block of the pair: planes hi and lo (TokTile)
  };
  struct alignas(16) Smem {
    Buf buf[2];
    T vt[NC][2][kTile][kTile];           // V rows of each state wave's columns
  };
};

template <int D>
constexpr int delta_pipe_threads() {
  return kWave * (4 + D / kTile);
}

template <typename T, int D, int F>
__global__ __launch_bounds__(delta_pipe_threads<D>()) void hyb_prefill_delta_pipe_kernel(
    PrefillArgs a, SegPlan pl) {
  typedef DeltaPipeCfg<T, D, F> C;
  typedef typename C::M M;
  typedef typename C::op_t op_t;
  typedef typename C::WFM WFM;
  typedef TokTile<2 * F> Tok;
  constexpr int f = C::f, E = M::E, KW = M::KW, NT = C::NT, NC = C::NC;
  static_assert(sizeof(T) == 2, "the pipelined increment is the bf16 path");
  static_assert(delta_pipe_threads<D>() == kWave * C::NWAVE, "launch bounds match the waves");
  __shared__ typename C::Smem sh;

  const int tid = threadIdx.x, lane = tid & (kWave - 1);
  const int w = __builtin_amdgcn_readfirstlane(tid / kWave);
  const int li = lane & 31, hh = lane >> 5;
  const int Hq = a.s.Hq, Hkv = a.s.Hkv, L = a.s.L, T_ = a.T;
  const int units = a.s.B * Hq;
  // pieces of segments 0 .. nseg-2 (the last segment's increment is never
  // needed)
  const int npc = pl.npieces();
  const int vix = xcd_unit(blockIdx.x, units * npc);
  const int u = vix % units, pc = vix / units;
  const int b = u / Hq, h = u % Hq, g = h / (Hq / Hkv);
  const int slot = a.slots ? a.slots[b] : b;
  if (slot < 0 || slot >= a.s.n_slots) return;  // uniform: no increment needed
  const size_t kstride = (size_t)Hkv * D;
  const int nblk = T_ / L;
  const int blk0 = pl.piece_lo(pc), blk1 = min(nblk, pl.piece_hi(pc));
  const int npair = max(0, (blk1 - blk0 + 1) / 2);
  const int nit = npair + 2;  // iterations -1 .. npair
  const bool row_ok = li < L;
  float* __restrict__ wsS = a.ws + ((size_t)u * npc + pc) * D * f;
  float* __restrict__ wsz = a.ws + (size_t)units * npc * D * f + ((size_t)u * npc + pc) * f;
  // Raw buffers over this request's rows of k and v (the launcher keeps a
  // request's rows under 2 GiB): a block's offset is a scalar.
  const __amdgpu_buffer_rsrc_t krs = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<T*>((const T*)a.k + (size_t)b * T_ * kstride), 0, (int)(T_ * kstride * sizeof(T)),
      kBufferWord3);
  const __amdgpu_buffer_rsrc_t vrs = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<T*>((const T*)a.v + (size_t)b * T_ * kstride), 0, (int)(T_ * kstride * sizeof(T)),
      kBufferWord3);
  auto koff = [&](int blk) { return (int)(((size_t)blk * L * kstride + (size_t)g * D) * sizeof(T)); };
  op_t ones;
#pragma unroll
  for (int e = 0; e < E; ++e) ones[e] = (T)1.0f;

  if (w < 4) {
    // ---- phi(K) of blocks blk0 + w + 4m: the first half in the iteration
    // before the block's pair is due, the second in the pair's iteration;
    // waves 2 and 3 idle in the first iteration, all after their last block,
    // so that every wave passes nit barriers ----
    constexpr float kLog2e = 1.4426950408889634f;
    constexpr int NA = NT * 8;  // second-sign exponentials in the first half
    op_t wop[NT][C::KD], x[C::KD];
    WFM::load_w((const T*)a.W + (size_t)h * F * D, li, hh, wop);
    // rows past the block length read row L-1 (finite); their phi is zeroed
    const int klane = (min(li, L - 1) * (int)kstride + hh * E) * (int)sizeof(T);
    auto load = [&](int blk) {
      const int so = koff(blk);
#pragma unroll
      for (int ks = 0; ks < C::KD; ++ks) x[ks] = buf_op<T>(krs, klane + ks * KW * (int)sizeof(T), so);
    };
    if (blk0 + w < blk1) load(blk0 + w);
    int nbar = 0;
    if (w >> 1) {
      lds_barrier();
      ++nbar;
    }
    for (int c = blk0 + w; c < blk1; c += 4) {
      // ---- first half ----
      float phi[C::NPAIR][16];
#pragma unroll
      for (int t = 0; t < NT; ++t) {
        f32x16 acc = {};
#pragma unroll
        for (int ks = 0; ks < C::KD; ++ks) acc = M::mma(wop[t][ks], x[ks], acc);
#pragma unroll
        for (int i = 0; i < 16; ++i) phi[t][i] = acc[i];
      }
      // (the operands are read by the products above before the rows of
      // this wave's next block land in the same registers)
      __builtin_amdgcn_sched_barrier(0);
      if (c + 4 < blk1) load(c + 4);
      float mx = -INFINITY, mn = INFINITY;
#pragma unroll
      for (int t = 0; t < NT; ++t)
#pragma unroll
        for (int i = 0; i < 16; ++i) {
          mx = fmaxf(mx, phi[t][i]);
          mn = fminf(mn, phi[t][i]);
        }
      mx = fmaxf(mx, xor32(mx));
      mn = fminf(mn, xor32(mn));
      // e^(u - mx) = 2^(u log2 e - mx log2 e): one fma per exponent; the
      // rounding of mx log2 e is common to the row and cancels in the ratio
      const float mxl = mx * kLog2e, mnl = mn * kLog2e;
      float sp = 0.0f, sn = 0.0f;
#pragma unroll
      for (int t = 0; t < NT; ++t)
#pragma unroll
        for (int i = 0; i < 16; ++i) {
          const float uu = phi[t][i];
          if (t * 16 + i < NA) {
            phi[NT + t][i] = __builtin_amdgcn_exp2f(__builtin_fmaf(-uu, kLog2e, mnl));
            sn += phi[NT + t][i];
          } else {
            phi[NT + t][i] = uu;
          }
          phi[t][i] = __builtin_amdgcn_exp2f(__builtin_fmaf(uu, kLog2e, -mxl));
          sp += phi[t][i];
        }
      lds_barrier();
      // ---- second half: the remaining exponentials, the sums,
      // normalisation (keep = row_ok zeroes a padding row) and the store ----
#pragma unroll
      for (int t = 0; t < NT; ++t)
#pragma unroll
        for (int i = 0; i < 16; ++i) {
          if (t * 16 + i < NA) continue;
          phi[NT + t][i] = __builtin_amdgcn_exp2f(__builtin_fmaf(-phi[NT + t][i], kLog2e, mnl));
          sn += phi[NT + t][i];
        }
      sp += xor32(sp);
      sn += xor32(sn);
      const float ip = row_ok ? 1.0f / sp : 0.0f, in = row_ok ? 1.0f / sn : 0.0f;
#pragma unroll
      for (int t = 0; t < NT; ++t)
#pragma unroll
        for (int i = 0; i < 16; ++i) {
          phi[t][i] *= ip;
          phi[NT + t][i] *= in;
        }
      const int j = (c - blk0) >> 1;
      char* kt = reinterpret_cast<char*>(sh.buf[j & 1].phiK[w & 1][0]);
      // (opaque: the piece addresses are formed here, not kept in registers
      // across the loop)
      int wb = Tok::write_base(li, hh);
      asm volatile("" : "+v"(wb));
#pragma unroll
      for (int p = 0; p < C::NPAIR; ++p)
#pragma unroll
        for (int i = 0; i < 16; i += 4) {  // features 32p + 2i + 4hh ..
          bf16x4 hi4, lo4;
          split_hi_lo4(&phi[p][i], hi4, lo4);
          const int at = wb ^ (16 * (4 * p + i / 4));
          *reinterpret_cast<bf16x4*>(kt + at) = hi4;
          *reinterpret_cast<bf16x4*>(kt + at + Tok::kPlane * 2) = lo4;
        }
      lds_barrier();
      nbar += 2;
    }
    for (; nbar < nit; ++nbar) lds_barrier();
  } else {
    // ---- state waves: commit pair i-1 in iteration i ----
    const int cw = w - 4, col = cw * kTile + li;
    f32x16 sacc[C::NRT];
#pragma unroll
    for (int rt = 0; rt < C::NRT; ++rt) sacc[rt] = f32x16{};
    // dz of the feature tiles cw, cw + NC, ... as accumulator tiles whose
    // columns are all equal: phi(K)^T 1 on the MFMAs
    f32x16 zt[C::ZPW];
#pragma unroll
    for (int j = 0; j < C::ZPW; ++j) zt[j] = f32x16{};
    // V rows of this wave's 32 columns for both blocks of a pair, an
    // iteration ahead: 4 lanes per row (16 bytes each), 16 rows per load; a
    // row at or past the block length reads past the buffer's end, as zeros
    int vlane[2];
#pragma unroll
    for (int s2 = 0; s2 < 2; ++s2) {
      const int t = s2 * 16 + (lane >> 2);
      vlane[s2] = t < L ? (t * (int)kstride + cw * kTile + (lane & 3) * 8) * (int)sizeof(T) : kPastBuffer;
    }
    op_t vrow[2][2];
    auto load_v = [&](int j) {
#pragma unroll
      for (int q = 0; q < 2; ++q) {
        const int so = koff(min(blk0 + 2 * j + q, blk1 - 1));
#pragma unroll
        for (int s2 = 0; s2 < 2; ++s2) vrow[q][s2] = buf_op<T>(vrs, vlane[s2], so);
      }
    };
    const int krb0 = Tok::read_base(lane);
    const T* vtr = &sh.vt[cw][0][4 * hh + ((lane & 15) >> 2)][16 * ((lane >> 4) & 1) + 4 * (lane & 3)];
    if (npair > 0) load_v(0);
    constexpr int RH = (C::NRT + 1) / 2;
    for (int i = -1; i <= npair; ++i) {
      const int j = i - 1;
      if (j >= 0 && j < npair) {
        typename C::Buf& B = sh.buf[j & 1];
        // V^T operands of the pair through this wave's LDS rows (its own
        // writes complete before its reads); the next pair's rows issued
#pragma unroll
        for (int q = 0; q < 2; ++q)
#pragma unroll
          for (int s2 = 0; s2 < 2; ++s2)
            *reinterpret_cast<op_t*>(&sh.vt[cw][q][s2 * 16 + (lane >> 2)][(lane & 3) * 8]) = vrow[q][s2];
        __builtin_amdgcn_sched_barrier(0);
        if (j + 1 < npair) load_v(j + 1);
        asm volatile("" ::: "memory");
        // read back transposed (lane li: column 32cw + li at the tokens
        // row_of(ks*E + e, hh))
        op_t vk[2][C::KL];
#pragma unroll
        for (int q = 0; q < 2; ++q)
#pragma unroll
          for (int ks = 0; ks < C::KL; ++ks)
            vk[q][ks] = lds_tr_op(vtr + (q * kTile + 16 * ks) * kTile, vtr + (q * kTile + 16 * ks + 8) * kTile);
        __builtin_amdgcn_sched_barrier(0);
        int krb = krb0;  // (opaque: the operand addresses are formed per pair)
        asm volatile("" : "+v"(krb));
        // LDS operands in batches ahead of their products (a scheduling
        // barrier after each batch): per block of the pair, the first half
        // of the row tiles, then the rest with z
#pragma unroll
        for (int q = 0; q < 2; ++q) {
          if (blk0 + 2 * j + q >= blk1) continue;  // uniform
          op_t kh[RH][C::KL], kl[RH][C::KL];
#pragma unroll
          for (int rt = 0; rt < RH; ++rt)
#pragma unroll
            for (int ks = 0; ks < C::KL; ++ks) {
              kh[rt][ks] = Tok::op(B.phiK[q][0], krb, rt, ks);
              kl[rt][ks] = Tok::op(B.phiK[q][1], krb, rt, ks);
            }
          __builtin_amdgcn_sched_barrier(0);
#pragma unroll
          for (int rt = 0; rt < RH; ++rt)
#pragma unroll
            for (int ks = 0; ks < C::KL; ++ks) {
              sacc[rt] = M::mma(kh[rt][ks], vk[q][ks], sacc[rt]);
              sacc[rt] = M::mma(kl[rt][ks], vk[q][ks], sacc[rt]);
            }
          __builtin_amdgcn_sched_barrier(0);
          op_t kh2[C::NRT - RH][C::KL], kl2[C::NRT - RH][C::KL], zh[C::ZPW][C::KL], zl[C::ZPW][C::KL];
#pragma unroll
          for (int rt = RH; rt < C::NRT; ++rt)
#pragma unroll
            for (int ks = 0; ks < C::KL; ++ks) {
              kh2[rt - RH][ks] = Tok::op(B.phiK[q][0], krb, rt, ks);
              kl2[rt - RH][ks] = Tok::op(B.phiK[q][1], krb, rt, ks);
            }
#pragma unroll
          for (int jz = 0; jz < C::ZPW; ++jz) {
            const int p = min(cw + jz * NC, C::NRT - 1);
#pragma unroll
            for (int ks = 0; ks < C::KL; ++ks) {
              zh[jz][ks] = Tok::op(B.phiK[q][0], krb, p, ks);
              zl[jz][ks] = Tok::op(B.phiK[q][1], krb, p, ks);
            }
          }
          __builtin_amdgcn_sched_barrier(0);
#pragma unroll
          for (int rt = RH; rt < C::NRT; ++rt)
#pragma unroll
            for (int ks = 0; ks < C::KL; ++ks) {
              sacc[rt] = M::mma(kh2[rt - RH][ks], vk[q][ks], sacc[rt]);
              sacc[rt] = M::mma(kl2[rt - RH][ks], vk[q][ks], sacc[rt]);
            }
#pragma unroll
          for (int jz = 0; jz < C::ZPW; ++jz) {
            const int p = cw + jz * NC;
            if (p >= C::NRT) continue;  // uniform
#pragma unroll
            for (int ks = 0; ks < C::KL; ++ks) {
              zt[jz] = M::mma(zh[jz][ks], ones, zt[jz]);
              zt[jz] = M::mma(zl[jz][ks], ones, zt[jz]);
            }
          }
        }
      }
      lds_barrier();
    }
#pragma unroll
    for (int rt = 0; rt < C::NRT; ++rt)
#pragma unroll
      for (int j = 0; j < 4; ++j)
        *reinterpret_cast<f32x4*>(wsS + (size_t)col * f + rt * kTile + row_of(4 * j, hh)) =
            f32x4{sacc[rt][4 * j], sacc[rt][4 * j + 1], sacc[rt][4 * j + 2], sacc[rt][4 * j + 3]};
#pragma unroll
    for (int j = 0; j < C::ZPW; ++j) {
      const int p = cw + j * NC;
      if (p < C::NRT && li == 0) {
#pragma unroll
        for (int i = 0; i < 16; i += 4)
          *reinterpret_cast<f32x4*>(wsz + p * kTile + row_of(i, hh)) =
              f32x4{zt[j][i], zt[j][i + 1], zt[j][i + 2], zt[j][i + 3]};
      }
    }
  }
}

template <typename T, int D, int F>
static hipError_t prefill_delta_go(const PrefillArgs& a, const SegPlan& p, hipStream_t st);

template <typename T, int D, int F>
static hipError_t prefill_go(const PrefillArgs& a, hipStream_t st) {
  const int units = a.s.B * a.s.Hq;
  const bool state_only = a.out == nullptr;
  const SegPlan p = state_only ? prefill_state_plan(a.s, a.T) : prefill_plan(a.s, a.T);
  const dim3 block(kWave * (D / kTile));
  if (p.nseg > 1) {
    const hipError_t e = prefill_delta_go<T, D, F>(a, p, st);
    if (e != hipSuccess) return e;
    const size_t per = (size_t)(D + 1) * 2 * F / 4;  // threads per unit
    const dim3 grid((unsigned)(units * ((per + 255) / 256)));
    if (state_only)
      hipLaunchKernelGGL(hyb_prefill_scan_kernel<true>, grid, dim3(256), 0, st, a, p);
    else
      hipLaunchKernelGGL(hyb_prefill_scan_kernel<false>, grid, dim3(256), 0, st, a, p);
    const hipError_t e0 = hipGetLastError();
    if (e0 != hipSuccess || state_only) return e0;
  }
  // The pipelined walk serves bf16 with F <= 64 when outputs are wanted;
  // the single-group walk serves the rest.
  if constexpr (sizeof(T) == 2 && F <= 64) {
    // (its buffer loads address a request's rows of q with 32-bit offsets)
    if (a.out != nullptr && (size_t)a.T * a.s.Hq * D * sizeof(T) < ((size_t)1 << 31)) {
      typedef PrefillPipeCfg<T, D, F> P;
      hipLaunchKernelGGL((hyb_prefill_pipe_kernel<T, D, F>), dim3(units * p.nseg),
                         dim3(kWave * P::NWAVE), 0, st, a, p);
      return hipGetLastError();
    }
  }
  hipLaunchKernelGGL((hyb_prefill_kernel<T, D, F>), dim3(units * p.nseg), block, 0, st, a, p, 0);
  return hipGetLastError();
}

template <typename T, int D, int F>
static hipError_t prefill_delta_go(const PrefillArgs& a, const SegPlan& p, hipStream_t st) {
  const int units = a.s.B * a.s.Hq;
  if (p.npieces() <= 0) return hipSuccess;
  if constexpr (sizeof(T) == 2 && F <= 64) {
    // (its buffer loads address a request's rows of k and v with 32-bit offsets)
    if ((size_t)a.T * a.s.Hkv * D * sizeof(T) < ((size_t)1 << 31)) {
      hipLaunchKernelGGL((hyb_prefill_delta_pipe_kernel<T, D, F>), dim3(units * p.npieces()),
                         dim3(delta_pipe_threads<D>()), 0, st, a, p);
      return hipGetLastError();
    }
  }
  hipLaunchKernelGGL((hyb_prefill_kernel<T, D, F>), dim3(units * p.npieces()),
                     dim3(kWave * (D / kTile)), 0, st, a, p, 1);
  return hipGetLastError();
}

template <typename T, int D>
static hipError_t prefill_delta_f(const PrefillArgs& a, const SegPlan& p, hipStream_t st) {
  switch (a.s.F) {
    case 32: return prefill_delta_go<T, D, 32>(a, p, st);
    case 64: return prefill_delta_go<T, D, 64>(a, p, st);
    case 128: return prefill_delta_go<T, D, 128>(a, p, st);
  }
  return hipErrorInvalidValue;
}

hipError_t launch_prefill_delta(const PrefillArgs& a, const SegPlan& p, hipStream_t st) {
  if (a.s.dtype == 1)
    return a.s.D == 64 ? prefill_delta_f<bf16, 64>(a, p, st) : prefill_delta_f<bf16, 128>(a, p, st);
  return a.s.D == 64 ? prefill_delta_f<float, 64>(a, p, st) : prefill_delta_f<float, 128>(a, p, st);
}


// One round of walk workgroups: a walk workgroup takes a whole CU (its LDS),
// so segments are what the batch's (request, head) units leave of 256 CUs to
// fill; at most 8 segments and at least 4 blocks per segment.  The increments
// of segments 0 .. nseg-2 are cut into pieces so that they too take about one
// workgroup per CU, with at least 2 blocks per piece (the increment kernel
// takes blocks in pairs).  The backward's walks use this plan as it is (they
// sum the pieces before or after their segment at their start); the prefill's
// workspace is sized by it.
SegPlan segment_plan(const Shape& s, int T) {
  constexpr int kCUs = 256;
  const int units = s.B * s.Hq, nblk = T / s.L;
  int nseg = (kCUs + units - 1) / units;
  if (nseg > 8) nseg = 8;
  if (nseg > nblk / 4) nseg = nblk / 4;
  if (nseg < 1) nseg = 1;
  for (; nseg > 1; --nseg)
    if ((nseg - 1) * ((nblk + nseg - 1) / nseg) < nblk) break;
  SegPlan p;
  p.nseg = nseg;
  p.sb = (nblk + nseg - 1) / nseg;
  p.ppseg = 1;
  p.pb = p.sb;
  if (nseg > 1) {
    int pp = (kCUs + units * (nseg - 1) - 1) / (units * (nseg - 1));
    if (pp > p.sb / 2) pp = p.sb / 2;
    if (pp < 1) pp = 1;
    // every piece non-empty
    for (; pp > 1; --pp)
      if ((pp - 1) * ((p.sb + pp - 1) / pp) < p.sb) break;
    p.ppseg = pp;
    p.pb = (p.sb + pp - 1) / pp;
  }
  return p;
}

// Workgroups of the walk and of the increments that the plan counts as one
// round.  One per CU for the pipelined kernels, by their LDS (106 KB of the walk's
// at d = f = 128; at d = f = 64, 59 and 41 KB, two would fit and are not counted),
// and for the single-group kernel at d = 128 by its registers (four waves of one
// per SIMD); two of it at d = 64.
static int prefill_fill(const Shape& s) {
  return s.dtype == 1 && s.F <= 64 ? 256 : s.D == 64 ? 512 : 256;
}

// Rounds of n workgroups of the given steps, in steps: workgroups that share a
// CU slow each other down (a third per neighbour).
static float prefill_rounds(long n, int fill, float steps) {
  const float share = (float)(n < fill ? n : fill) / 256.0f;
  return (float)((n + fill - 1) / fill) * steps * (share > 1.0f ? 0.67f + 0.33f * share : 1.0f);
}

// The prefill's plan: the (segments, pieces per segment) with the least
// estimated time among those whose pieces fit the workspace of segment_plan.
// In walk steps: rounds of walk workgroups times a segment's blocks and its
// start; rounds of increment workgroups times a piece's blocks, at 0.45 of a step
// each, and their start; and the two launches.  A start takes about 4 and 2 steps
// of the pipelined kernels (2 to 3 us each) and the launches 4; of the
// single-group kernel's steps (10 to 37 us) a start takes 1 or half, the launches
// half.  (Priced like the pipelined kernels' a prompt of 256 tokens was not cut:
// fp32 302 us, 205 so; f = 256 127, 96 so.)
// (Counting two of the fp32 kernel's workgroups per CU at d = 128, where its
// registers let one in, took 4 x 2048 tokens from 1112 to 1318 us; as counted
// here they take 1069 us.)
// With up to 8 segments, as the backward's, one prompt of 16384 tokens walks
// on 128 CUs: 240 us, against 126 us with the 16 segments chosen here (2 of
// 8192: 162 and 125, 4 of 2048: 99 and 79, 1 of 1024: 66 and 35).
SegPlan prefill_plan(const Shape& s, int T) {
  const int units = s.B * s.Hq, nblk = T / s.L, room = segment_plan(s, T).npieces();
  const int fill = prefill_fill(s);
  const bool pipe = s.dtype == 1 && s.F <= 64;
  const float start = pipe ? 4.0f : 1.0f, extra = pipe ? 4.0f : 0.5f;
  SegPlan best;
  best.sb = best.pb = nblk;
  float least = prefill_rounds(units, fill, (float)nblk + start);
  SegPlan p;
  for (p.nseg = 2; p.nseg <= room + 1 && p.nseg <= nblk; ++p.nseg) {
    p.sb = (nblk + p.nseg - 1) / p.nseg;
    if ((p.nseg - 1) * p.sb >= nblk) continue;  // the last segment non-empty
    for (p.ppseg = 1; p.npieces() <= room && p.ppseg <= p.sb; ++p.ppseg) {
      p.pb = (p.sb + p.ppseg - 1) / p.ppseg;
      if ((p.ppseg - 1) * p.pb >= p.sb) continue;  // every piece non-empty
      const long wg = (long)units * p.nseg, dg = (long)units * p.npieces();
      const float cost = prefill_rounds(wg, fill, (float)p.sb + start) +
                         prefill_rounds(dg, fill, 0.45f * (float)p.pb + 0.5f * start) + extra;
      if (cost < least) {
        least = cost;
        best = p;
      }
    }
  }
  return best;
}

// The plan without outputs: pieces over the whole prompt (segments 0 ..
// nseg-2 of a plan whose last segment is empty), as many as fit the workspace
// and the chip in one round, of at least 2 blocks; nseg = 1 (one walk per
// unit) where there is no workspace.  16384 tokens: 42 us, against 297 us
// when the last segment still walked, on the unit's one workgroup (8 prompts
// of 8192: 138 and 476).
SegPlan prefill_state_plan(const Shape& s, int T) {
  const int units = s.B * s.Hq, nblk = T / s.L, room = segment_plan(s, T).npieces();
  SegPlan p;
  p.sb = p.pb = nblk;
  if (room < 1) return p;
  int n = prefill_fill(s) / units;
  n = n > room ? room : n;
  n = n < 1 ? 1 : n;
  p.sb = p.pb = (nblk + n - 1) / n < 2 ? 2 : (nblk + n - 1) / n;
  p.nseg = (nblk + p.sb - 1) / p.sb + 1;
  return p;
}

size_t prefill_delta_ws_bytes(const Shape& s, const SegPlan& p) {
  if (p.npieces() <= 0) return 0;
  const size_t f = 2 * (size_t)s.F;
  return (size_t)s.B * s.Hq * p.npieces() * ((size_t)s.D * f + f) * 4;
}

size_t prefill_ws_bytes(const Shape& s, int T) {
  const SegPlan p = segment_plan(s, T);
  if (p.nseg <= 1) return 0;
  const size_t f = 2 * (size_t)s.F;
  // the increments, then the incoming state
  return prefill_delta_ws_bytes(s, p) + (size_t)s.B * s.Hq * ((size_t)s.D * f + f) * 4;
}

template <typename T, int D>
static hipError_t prefill_f(const PrefillArgs& a, hipStream_t st) {
  switch (a.s.F) {
    case 32: return prefill_go<T, D, 32>(a, st);
    case 64: return prefill_go<T, D, 64>(a, st);
    case 128: return prefill_go<T, D, 128>(a, st);
  }
  return hipErrorInvalidValue;
}

template <typename T>
static hipError_t prefill_d(const PrefillArgs& a, hipStream_t st) {
  switch (a.s.D) {
    case 64: return prefill_f<T, 64>(a, st);
    case 128: return prefill_f<T, 128>(a, st);
  }
  return hipErrorInvalidValue;
}

hipError_t launch_prefill(const PrefillArgs& a, hipStream_t st) {
  return a.s.dtype == 1 ? prefill_d<bf16>(a, st) : prefill_d<float>(a, st);
}

}  // namespace hyb
