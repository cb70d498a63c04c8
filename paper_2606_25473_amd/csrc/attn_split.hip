// attn_split.hip -- bf16 masked attention forward + JVP for launches with few query tiles.
//
// The kernels of attn_mfma.hip give each work-group 256 (JVP) or 128 (forward) query rows and
// all their keys.  A launch with fewer such tiles than the chip has CUs leaves the others
// idle, and its time is the longest tile's serial walk over the keys.  Here the 8 waves of a
// work-group form RG row groups of 32 query rows and KS key splits: wave (rg, ks) walks the
// blocks ks, ks + KS, ... of its tile's plan (schedule.hpp) with its own running max,
// normaliser and accumulators, and the KS partial results of a row are merged through LDS at
// the end (the online-softmax merge, in a fixed order: results are deterministic and need no
// memory beyond the outputs).  A tile has KS times fewer rows and KS times fewer steps, so a
// launch has KS times as many work-groups, each KS times shorter.
//
// What bounds it: per key block and wave the matrix work is that of attn_mfma.hip, but a
// block staged in LDS serves RG waves instead of 8, so the traffic from L2 grows 8 / RG
// times; that is why full launches keep the larger tiles (choose_ksplit in layout.cpp).
//
// LDS holds one key block per split and stage, in two stages where they fit (the next round's
// blocks stream in while a round is computed, one barrier per round).  The D = 128 JVP with
// four splits would need 256 KiB for that: it has one stage.  K and dK are read in the score
// phase only, V and dV in the output phase only, so the next K, dK stream in during the output
// phase and the next V, dV during the score phase, with a barrier after each phase.
//
// Forward, JVP and zero-clean JVP use the same tiles, splits and merge order, so that their
// outputs agree bit for bit wherever the mathematics says they are equal.
#include <hip/hip_runtime.h>

#include <stdint.h>

#include "kernels.hpp"
#include "mfma_common.hpp"

namespace attn {
namespace {

using namespace dev;

constexpr int BC = kMfmaBc;
constexpr float kLazy = 8.0f;
constexpr int NW = 8;

enum { kFwd = 0, kJvp = 1, kZeroClean = 2 };

template <bool B>
struct Tag {
  static constexpr bool value = B;
};

template <int D, int MODE, int KS>
struct SGeo {
  static constexpr bool JVP = MODE != kFwd;
  static constexpr int RG = NW / KS;              // row groups of 32 query rows
  static constexpr int BR = 32 * RG;              // query rows per work-group
  static constexpr int ROWB = D * 2;              // bytes per LDS row
  static constexpr int TILEB = BC * ROWB;         // one tile of BC keys
  static constexpr int DT = D / 32;
  static constexpr int KSTEPS = D / 16;           // 16-deep k steps of the score contraction
  static constexpr int IPT = TILEB / 1024;        // 1 KiB direct loads per tile
  static constexpr int NS = 16 * DT;              // accumulator slots per lane
  static constexpr int OWN = NS / KS;             // slots a wave merges and stores
  static constexpr int STB = (JVP ? 4 : 2) * KS * TILEB;  // a stage: one block of every split
  static constexpr int DQB = JVP ? BR * ROWB : 0;
  static constexpr int NST = 2 * STB + DQB <= 160 * 1024 ? 2 : 1;
  static constexpr int XCHG = NW * NS * 64 * 4;   // one accumulator set of every wave, fp32
  static constexpr int STATS = NW * 32 * 4 * 4;   // m, l, r of every wave's rows
  static constexpr int LOOP = NST * STB + DQB, MERGE = XCHG + STATS;
  static constexpr int BYTES = LOOP > MERGE ? LOOP : MERGE;
  static_assert(IPT % RG == 0 && OWN % 4 == 0, "whole loads per wave, whole 4-value stores");
  static_assert(BYTES <= 160 * 1024, "LDS of a CU");
};

template <int D, int MODE, int KS>
__device__ __forceinline__ void split_body(const AttnArgs& a, const int bh, const int qtile, char* const lds) {
  using G = SGeo<D, MODE, KS>;
  constexpr bool JVP = G::JVP, ZC = MODE == kZeroClean;
  constexpr int TB = G::TILEB, RG = G::RG;
  constexpr int KB = 0, VB = KS * TB, DKB = 2 * KS * TB, DVB = 3 * KS * TB;  // within a stage
  constexpr int QB = G::NST * G::STB;

  const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
  const int lane = threadIdx.x & 63;
  const int hh = lane >> 5;
  const int rg = wave % RG, ks = wave / RG;
  const int L = a.L;
  const int t0 = ZC ? a.t0 : 0;  // tangent rows are [t0, L)
  const int Lt = L - t0;

  const size_t head = (size_t)bh * L * D;
  const size_t thead = (size_t)bh * Lt * D;
  const bf16_t* __restrict__ Qg = (const bf16_t*)a.Q + head;
  const bf16_t* __restrict__ Kg = (const bf16_t*)a.K + head;
  const bf16_t* __restrict__ Vg = (const bf16_t*)a.V + head;
  const bf16_t* __restrict__ dQg = (const bf16_t*)a.dQ + thead;
  const bf16_t* __restrict__ dKg = (const bf16_t*)a.dK + thead;
  const bf16_t* __restrict__ dVg = (const bf16_t*)a.dV + thead;

  int q0, q1;  // (the tile may be cut at a group bound: its rows end at q1)
  tile_rows(a.order, qtile, G::BR, L, &q0, &q1);
  const TilePlan plan = plan_tile(a.gt, q0, q1, BC);
  const int nblk = plan_num_blocks(plan);
  const int niter = (nblk + KS - 1) / KS;
  // (kZeroClean) the plan visits key blocks in increasing order, so the first ja rounds hold
  // no tangent keys at all: they load no dK, dV and drop those products.  From round ja on
  // every block has its tangent tiles, with the rows below t0 cleared.
  const int ja = ZC ? imin(plan_blocks_below(plan, t0 / BC) / KS, niter) : 0;

  const int qrow = rg * 32 + (lane & 31);
  const int row = q0 + qrow;
  const int wrow0 = imin(q0 + rg * 32, q1 - 1);
  const WaveRanges wr = wave_ranges(a.gt, wrow0, imin(wrow0 + 31, q1 - 1));

  // Q^T as B operand (lane: row l%32, d = 16 s + 8 (l/32) + 0..7); rows past the end are
  // clamped to the last row (their outputs are not stored)
  bf16x8 qop[G::KSTEPS];
#pragma unroll
  for (int s = 0; s < G::KSTEPS; ++s) qop[s] = *(const bf16x8*)(Qg + (size_t)imin(row, L - 1) * D + 16 * s + 8 * hh);

  // ---- direct loads: one instruction moves 1 KiB (RPI rows); the XOR swizzle is applied by
  // choosing the chunk each lane fetches; rows past the end are clamped to the last one
  constexpr int RPI = 1024 / G::ROWB;
  const int dma_r = (lane * 16) / G::ROWB;
  const int dma_phys = ((lane * 16) % G::ROWB) >> 4;
  const unsigned lds0 = __builtin_amdgcn_readfirstlane(lds_addr(lds));
  auto dma_rows = [&](const bf16_t* src, int row0, int r, unsigned dst) {
    const int rr = r + dma_r;
    const unsigned grow = (unsigned)imin(row0 + rr, L - 1);
    lds_load16(src, (grow * D + (unsigned)((dma_phys ^ swz<D>(rr)) * 8)) * 2u, dst + (unsigned)(r * G::ROWB));
  };
  // sequence row x is tangent row x - t0; rows below t0 are clamped to tangent row 0 and
  // cleared in LDS (clear_t) before anyone reads them
  auto dma_rows_t = [&](const bf16_t* src, int row0, int r, unsigned dst) {
    const int rr = r + dma_r;
    const unsigned grow = (unsigned)imin(imax(row0 + rr - t0, 0), Lt - 1);
    lds_load16(src, (grow * D + (unsigned)((dma_phys ^ swz<D>(rr)) * 8)) * 2u, dst + (unsigned)(r * G::ROWB));
  };
  // The RG waves of a split share its block's loads: wave rg issues instructions
  // [rg IPT / RG, (rg + 1) IPT / RG) of each tile.
  constexpr int IPW = G::IPT / RG;
  const unsigned own = lds0 + (unsigned)(ks * TB);  // this split's tile within each buffer
  auto load = [&](const bf16_t* src, const bf16_t* tsrc, int i, unsigned off, unsigned toff) {  // (off, toff: in LDS)
    if (i >= nblk) return;
    const int k0 = plan_block(plan, i) * BC;
#pragma unroll
    for (int j = 0; j < IPW; ++j) dma_rows(src, k0, (rg * IPW + j) * RPI, own + off);
    if constexpr (JVP) {
      if (!ZC || i >= ja * KS) {
#pragma unroll
        for (int j = 0; j < IPW; ++j) dma_rows_t(tsrc, k0, (rg * IPW + j) * RPI, own + toff);
      }
    }
  };
  // tangent rows below t0: each lane clears the 16-byte pieces that it loaded itself (its own
  // loads have landed, the barrier is still ahead)
  auto clear_t = [&](int row0, int r, unsigned dst) {
    if (row0 + r + dma_r < t0) *(__attribute__((address_space(3))) u32x4*)(uintptr_t)(dst + r * G::ROWB + lane * 16) = u32x4{0u, 0u, 0u, 0u};
  };
  auto clear_block = [&](int i, unsigned toff) {
    if constexpr (ZC) {
      if (i >= ja * KS && i < nblk) {
        const int k0 = plan_block(plan, i) * BC;
        if (k0 < t0) {
#pragma unroll
          for (int j = 0; j < IPW; ++j) clear_t(k0, (rg * IPW + j) * RPI, own + toff);
        }
      }
    }
  };
  auto sync = []() { asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier" ::: "memory"); };
  auto landed = []() { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); };

  // ---- per-lane operand offsets (lds_off(row, chunk) ^ 32 s; see tr_bases)
  unsigned trx[2];
  tr_bases<D>(lane, trx);
  const unsigned koff = lds_off<D>(lane & 31, hh), dqoff = lds_off<D>(qrow, hh);

  f32x16 oacc[G::DT], tacc[JVP ? G::DT : 1];
#pragma unroll
  for (int dt = 0; dt < G::DT; ++dt) {
    oacc[dt] = f32x16{};
    if constexpr (JVP) tacc[dt] = f32x16{};
  }
  float m = -INFINITY, lsum = 0.f, rsum = 0.f;
  const float c2 = a.scale * kLog2e;
  const float sc = a.scale;

  // ---- prologue: dQ of the tile, the first block of every split
  if constexpr (JVP) {
    constexpr int IPQ = G::BR * G::ROWB / 1024;
#pragma unroll
    for (int j0 = 0; j0 < IPQ; j0 += NW)
      if (IPQ % NW == 0 || j0 + wave < IPQ) dma_rows_t(dQg, q0, (j0 + wave) * RPI, lds0 + QB);
  }
  load(Kg, dKg, ks, KB, DKB);
  load(Vg, dVg, ks, VB, DVB);
  __builtin_amdgcn_s_waitcnt(0xF70);  // vmcnt(0), known to the compiler: also the Q operands
  landed();
  if constexpr (ZC) {
    if (q0 < t0) {
      constexpr int IPQ = G::BR * G::ROWB / 1024;
#pragma unroll
      for (int j0 = 0; j0 < IPQ; j0 += NW)
        if (IPQ % NW == 0 || j0 + wave < IPQ) clear_t(q0, (j0 + wave) * RPI, lds0 + QB);
    }
    clear_block(ks, DKB);
    clear_block(ks, DVB);
  }
  sync();

  // The reference max of every split from the first block, as the unsplit kernels take it: P~ is
  // then rounded against the same reference for any number of splits, and the results differ from
  // theirs by the order of the fp32 sums alone (forward, 12 heads, D = 64, full, L = 1560, against
  // full tiles: rel-L2 4.6e-5 instead of 2.5e-3; the time is the same).  Rows that the first block
  // does not admit take each split's own, below, and so do waves that span many groups, where one
  // more mask costs up to 5 us.
  if (nblk > 0 && wr.direct) {
    const BlockMask mask = block_mask(a.gt, wr, plan, row, plan_block(plan, 0) * BC, L);
    if (!mask.none) {
      f32x16 S = f32x16{};
#pragma unroll
      for (int s = 0; s < G::KSTEPS; ++s) S = mfma(ld128_at((lds0 + KB + koff) ^ (32u * s)), qop[s], S);
      float sv[16];
      const uint32_t bits = mask.bits >> (4 * hh);
#pragma unroll
      for (int e = 0; e < 16; ++e) sv[e] = (bits >> (8 * (e >> 2) + (e & 3))) & 1u ? S[e] : -INFINITY;
      const float mloc = max16(sv) * c2, mx = fmaxf(mloc, xor32(mloc));
      if (mx > m) m = mx;
    }
  }

  // one round: KS consecutive blocks of the plan, one per split; TK: with tangent keys
  auto round = [&](auto tk, const int j) {
    constexpr bool TK = JVP && decltype(tk)::value;
    const int i = j * KS + ks;
    // this round's stage, and the one that the next round's loads fill
    const unsigned cur = G::NST == 2 ? (unsigned)((j & 1) * G::STB) : 0u;
    const unsigned nxt = G::NST == 2 ? (unsigned)(G::STB - (j & 1) * G::STB) : 0u;
    if constexpr (G::NST == 2) {
      load(Kg, dKg, i + KS, nxt + KB, nxt + DKB);
      load(Vg, dVg, i + KS, nxt + VB, nxt + DVB);
    }
    // (uniform) the last round may leave some splits idle, and a tile that spans groups visits
    // the union of its rows' blocks, some of which this wave's rows do not see at all
    bool active = i < nblk;
    BlockMask mask{};
    if (active) {
      mask = block_mask(a.gt, wr, plan, row, plan_block(plan, i) * BC, L);
      active = !mask.none;
    }
    f32x16 S = f32x16{}, dS = f32x16{};

    // ---- S^T = K Q^T, dS^T = dK Q^T + K dQ^T, operands read one k step ahead
    if (active) {
      const unsigned kb = vreg_add(own + cur + KB, koff, j), qb = vreg_add(lds0 + QB, dqoff, j);
      constexpr int SPF = JVP ? 1 : 2;
      bf16x8 kop[SPF + 1], dkop[SPF + 1], dqop[SPF + 1];
      auto read = [&](int s) {
        const int b = s % (SPF + 1);
        kop[b] = ld128_at(kb ^ (32u * s));
        if constexpr (TK) dkop[b] = ld128_at((kb ^ (32u * s)) + (DKB - KB));
        if constexpr (JVP) dqop[b] = ld128_at(qb ^ (32u * s));
      };
#pragma unroll
      for (int s = 0; s < SPF; ++s) read(s);
#pragma unroll
      for (int s = 0; s < G::KSTEPS; ++s) {
        if (s + SPF < G::KSTEPS) read(s + SPF);
        __builtin_amdgcn_sched_barrier(0);
        const int b = s % (SPF + 1);
        S = mfma(kop[b], qop[s], S);
        if constexpr (TK) dS = mfma(dkop[b], qop[s], dS);
        if constexpr (JVP) dS = mfma(kop[b], dqop[b], dS);
        __builtin_amdgcn_sched_barrier(0);
      }
    }
    // (one stage) every wave is done with K, dK of round j, and V, dV of round j have landed
    if constexpr (G::NST == 1) {
      if constexpr (ZC) {
        landed();
        if (j > 0) clear_block(i, DVB);
      }
      sync();
      load(Kg, dKg, i + KS, KB, DKB);
    }

    if (active) {
      float sv[16], dsv[16];
#pragma unroll
      for (int e = 0; e < 16; ++e) {
        sv[e] = S[e];
        dsv[e] = JVP ? dS[e] : 0.f;
      }
      if (!mask.all) {
        const uint32_t bits = mask.bits >> (4 * hh);
#pragma unroll
        for (int e = 0; e < 16; ++e) {
          const bool ok = (bits >> (8 * (e >> 2) + (e & 3))) & 1u;
          sv[e] = ok ? sv[e] : -INFINITY;
          dsv[e] = ok ? dsv[e] : 0.f;
        }
      }
      // online softmax; the reference max moves only when a row's block max exceeds it by
      // more than kLazy (log2 units)
      const float mloc = max16(sv) * c2;
      if (__ballot(mloc > m + kLazy) != 0) {
        const float mx = fmaxf(mloc, xor32(mloc));
        const bool up = mx > m + kLazy;
        const float mnew = up ? mx : m;
        const float alpha = up ? __builtin_amdgcn_exp2f(m - mnew) : 1.f;
        lsum *= alpha;
        if constexpr (JVP) rsum *= alpha;
#pragma unroll
        for (int dt = 0; dt < G::DT; ++dt) {
          oacc[dt] *= alpha;
          if constexpr (JVP) tacc[dt] *= alpha;
        }
        m = mnew;
      }
      const float mneg = m == -INFINITY ? 0.f : -m;
      float p[16];
#pragma unroll
      for (int e = 0; e < 16; ++e) {
        p[e] = __builtin_amdgcn_exp2f(fmaf(sv[e], c2, mneg));
        lsum += p[e];
      }
      bf16x8 pb[2], hb[2];
#pragma unroll
      for (int t = 0; t < 2; ++t)
#pragma unroll
        for (int e = 0; e < 8; ++e) pb[t][e] = (bf16_t)p[8 * t + e];
      if constexpr (JVP) {
#pragma unroll
        for (int e = 0; e < 16; ++e) {
          const float hv = p[e] * (dsv[e] * sc);
          rsum += hv;
          hb[e >> 3][e & 7] = (bf16_t)hv;
        }
      }

      // ---- O^T += V^T P~^T ; T^T += dV^T P~^T + V^T H~^T
      constexpr int OPF = JVP ? 1 : 2;
      constexpr int NG = 2 * G::DT;
      const unsigned vb0 = vreg_add(own + cur + VB, trx[0], j), vb1 = vreg_add(own + cur + VB, trx[1], j);
      bf16x8 vop[OPF + 1], dvop[OPF + 1];
      auto read = [&](int g) {
        const int t = g / G::DT, dt = g % G::DT, b = g % (OPF + 1);
        const unsigned o = 16u * t * G::ROWB;
        const unsigned a0 = (vb0 ^ (64u * dt)) + o, a1 = (vb1 ^ (64u * dt)) + o;
        vop[b] = cat(ld_tr_at(a0), ld_tr_at(a1));
        if constexpr (TK) dvop[b] = cat(ld_tr_at(a0 + (DVB - VB)), ld_tr_at(a1 + (DVB - VB)));
      };
#pragma unroll
      for (int g = 0; g < OPF; ++g) read(g);
#pragma unroll
      for (int g = 0; g < NG; ++g) {
        if (g + OPF < NG) read(g + OPF);
        __builtin_amdgcn_sched_barrier(0);
        const int t = g / G::DT, dt = g % G::DT, b = g % (OPF + 1);
        oacc[dt] = mfma(vop[b], pb[t], oacc[dt]);
        if constexpr (TK) tacc[dt] = mfma(dvop[b], pb[t], tacc[dt]);
        if constexpr (JVP) tacc[dt] = mfma(vop[b], hb[t], tacc[dt]);
        __builtin_amdgcn_sched_barrier(0);
      }
    }
    // every wave is done with round j (one stage: with its V, dV), and the loads for round
    // j + 1 (one stage: its K, dK) have landed
    if constexpr (ZC) {
      landed();
      clear_block(i + KS, nxt + DKB);
      if constexpr (G::NST == 2) clear_block(i + KS, nxt + DVB);
    }
    sync();
    if constexpr (G::NST == 1) load(Vg, dVg, i + KS, VB, DVB);
  };
  int j = 0;
  if constexpr (ZC)
    for (; j < ja; ++j) round(Tag<false>{}, j);
  for (; j < niter; ++j) round(Tag<true>{}, j);

  // ---- merge the KS partial results of each row (no load is in flight: the last round
  // issued none).  With M the largest reference max, split s enters with weight
  // 2^(m_s - M); a split that saw no key of the row has l = 0 (and where the first block gave it
  // no reference either, m = -inf and weight 0).
  float* const st = (float*)(lds + G::XCHG);
  const float lt = lsum + xor32(lsum);
  const float rt = JVP ? rsum + xor32(rsum) : 0.f;
  if (hh == 0) *(float4*)(st + (wave * 32 + lane) * 4) = make_float4(m, lt, rt, 0.f);
  float* const xo = (float*)lds + (size_t)wave * G::NS * 64 + lane;
#pragma unroll
  for (int e = 0; e < G::NS; ++e) xo[e * 64] = oacc[e >> 4][e & 15];
  __syncthreads();
  float wgt[KS], l_tot = 0.f, r_tot = 0.f, M = -INFINITY;
  float4 sv4[KS];
#pragma unroll
  for (int s = 0; s < KS; ++s) {
    sv4[s] = *(const float4*)(st + ((s * RG + rg) * 32 + (lane & 31)) * 4);
    M = fmaxf(M, sv4[s].x);
  }
#pragma unroll
  for (int s = 0; s < KS; ++s) {
    wgt[s] = sv4[s].x == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(sv4[s].x - M);
    l_tot = fmaf(wgt[s], sv4[s].y, l_tot);
    r_tot = fmaf(wgt[s], sv4[s].z, r_tot);
  }
  const float inv = l_tot > 0.f ? 1.f / l_tot : 0.f;
  // this wave's OWN slots of every split: slot e holds d = 32 (e / 16) + 8 (e%16 / 4) + 4 hh + e%4
  auto merged = [&](float (&out)[G::OWN]) {
#pragma unroll
    for (int e = 0; e < G::OWN; ++e) {
      float v = 0.f;
#pragma unroll
      for (int s = 0; s < KS; ++s)
        v = fmaf(wgt[s], ((const float*)lds)[((size_t)(s * RG + rg) * G::NS + ks * G::OWN + e) * 64 + lane], v);
      out[e] = v;
    }
  };
  auto store = [&](bf16_t* dst, const float (&v)[G::OWN]) {
#pragma unroll
    for (int c = 0; c < G::OWN / 4; ++c) {
      const int q4 = ks * (G::OWN / 4) + c;  // which run of 4 slots
      bf16x4 o;
#pragma unroll
      for (int e = 0; e < 4; ++e) o[e] = (bf16_t)v[4 * c + e];
      *(bf16x4*)(dst + 8 * q4 + 4 * hh) = o;
    }
  };
  float on[G::OWN];
  merged(on);
#pragma unroll
  for (int e = 0; e < G::OWN; ++e) on[e] *= inv;
  if (row < q1) {
    store((bf16_t*)a.O + head + (size_t)row * D, on);
    if (hh == 0 && ks == 0) a.LSE[(size_t)bh * L + row] = l_tot > 0.f ? (M + __log2f(l_tot)) * kLn2 : -INFINITY;
  }
  if constexpr (JVP) {
    __syncthreads();
#pragma unroll
    for (int e = 0; e < G::NS; ++e) xo[e * 64] = tacc[e >> 4][e & 15];
    __syncthreads();
    float tn[G::OWN];
    merged(tn);
#pragma unroll
    for (int e = 0; e < G::OWN; ++e) tn[e] = (tn[e] - r_tot * on[e]) * inv;
    // (zero-clean: dO of rows below t0 is zero and not stored)
    if (row < q1 && row >= t0) store((bf16_t*)a.dO + thead + (size_t)(row - t0) * D, tn);
  }
}

template <int D, int MODE, int KS>
__global__ __launch_bounds__(64 * NW) __attribute__((amdgpu_waves_per_eu(2, 2)))
void attn_split_kernel(const AttnArgs a) {
  using G = SGeo<D, MODE, KS>;
  static_assert(int(SGeo<D, kFwd, KS>::BYTES) <= int(G::BYTES), "the zero-clean kernel also runs the forward body");
  __shared__ __attribute__((aligned(1024))) char lds[G::BYTES];
  const TileSlot sl = slot_of(blockIdx.x, a.B * a.H, a.order.nt, kHeadGroup);
  const int qtile = tile_of(a.order, sl.pos);
  if constexpr (MODE == kZeroClean) {
    int q0, q1;
    tile_rows(a.order, qtile, G::BR, a.L, &q0, &q1);
    if (q1 <= a.t0) {  // no tangent row in the tile: the primal only
      split_body<D, kFwd, KS>(a, sl.bh, qtile, lds);
      return;
    }
  }
  split_body<D, MODE, KS>(a, sl.bh, qtile, lds);
}

template <int D, int KS>
void launch(const AttnArgs& a, Pass pass, const dim3& grid, hipStream_t stream) {
  const dim3 block(64 * NW);
  if (pass == Pass::kJvp) hipLaunchKernelGGL((attn_split_kernel<D, kJvp, KS>), grid, block, 0, stream, a);
  else if (pass == Pass::kJvpZeroClean)
    hipLaunchKernelGGL((attn_split_kernel<D, kZeroClean, KS>), grid, block, 0, stream, a);
  else hipLaunchKernelGGL((attn_split_kernel<D, kFwd, KS>), grid, block, 0, stream, a);
}

}  // namespace

hipError_t launch_split_bf16(const AttnArgs& a, int D, Pass pass, hipStream_t stream) {
  const dim3 grid((unsigned)(a.order.nt * a.B * a.H));
  if (D == 128) a.ksplit == 4 ? launch<128, 4>(a, pass, grid, stream) : launch<128, 2>(a, pass, grid, stream);
  else a.ksplit == 4 ? launch<64, 4>(a, pass, grid, stream) : launch<64, 2>(a, pass, grid, stream);
  return hipGetLastError();
}

}  // namespace attn
