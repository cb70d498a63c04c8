// attn_bwd_split.hip -- bf16 masked attention backward for launches with few tiles.
//
// The passes of attn_bwd.hip give a work-group 256 query rows or 128 keys; a launch with fewer
// such tiles than CUs leaves the others idle.  Here, as in attn_split.hip, the 8 waves of a
// work-group form row (key) groups of 32 and splits of the other side: split s walks the
// blocks s, s + splits, ... of the tile's plan, and the splits' partial gradients are summed
// through LDS at the end in a fixed order (deterministic, no memory beyond the outputs).
//  - query-tile pass: KS key splits, 256 / KS rows per tile, 32 keys per split and round;
//  - key-tile pass: 4 query splits, 64 keys per tile, 32 query rows per split and round.
// Both stage one block per split in LDS, in two stages (the next round's blocks stream in
// while a round is computed, one barrier per round).  Per block and wave the matrix work and
// the operand reads are those of attn_bwd.hip; the L2 traffic grows with the splits, so full
// launches keep the larger tiles (choose_bwd_ksplit, choose_qsplit in layout.cpp).
#include <hip/hip_runtime.h>

#include <stdint.h>

#include "kernels.hpp"
#include "mfma_common.hpp"

namespace attn {
namespace {

using namespace dev;

constexpr int NW = 8;
constexpr int NTHREADS = 64 * NW;
constexpr int BC = 32;  // keys (query rows) per block

__device__ __forceinline__ void sync_all() { asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier" ::: "memory"); }

// N splits, 8 / N groups of 32 rows (keys) per work-group
template <int D, int N>
struct SGeo {
  static constexpr int RG = NW / N;
  static constexpr int BR = 32 * RG;
  static constexpr int ROWB = D * 2;
  static constexpr int TILEB = BC * ROWB;
  static constexpr int DT = D / 32;
  static constexpr int KSTEPS = D / 16;
  static constexpr int IPT = TILEB / 1024;
  static constexpr int IPW = IPT / RG;           // direct loads per wave and tile
  static constexpr int NS = 16 * DT;             // accumulator slots per lane
  static constexpr int OWN = NS / N;             // slots a wave sums and stores
  static constexpr int XCHG = NW * NS * 64 * 4;  // one accumulator set of every wave
  static_assert(IPT % RG == 0 && OWN % 4 == 0, "whole loads per wave, whole 4-value stores");
};

// Direct loads of one 32-row block into the LDS tile at dst, instructions [j0, j0 + n) of the
// tile by this wave (1 KiB each); the XOR swizzle picks the chunk each lane fetches; rows past
// the end are clamped to the last one.
template <int D, int N>
__device__ __forceinline__ void load_rows(const bf16_t* src, int row0, int L, int j0, unsigned dst, int lane) {
  constexpr int ROWB = 2 * D, RPI = 1024 / ROWB;
  const int r = (lane * 16) / ROWB, phys = ((lane * 16) % ROWB) >> 4;
#pragma unroll
  for (int j = 0; j < N; ++j) {
    const int rr = (j0 + j) * RPI + r;
    const unsigned grow = (unsigned)imin(row0 + rr, L - 1);
    lds_load16(src, (grow * D + (unsigned)((phys ^ swz<D>(rr)) * 8)) * 2u, dst + (unsigned)((j0 + j) * 1024));
  }
}

// Sum over the splits of this wave's OWN slots, from the exchange area (wave (rg, s) at index
// s RG + rg, slots of 64 lanes).
template <class G, int N>
__device__ __forceinline__ void put(float* x, int wave, int lane, const f32x16 (&acc)[G::DT]) {
  float* const o = x + (size_t)wave * G::NS * 64 + lane;
#pragma unroll
  for (int e = 0; e < G::NS; ++e) o[e * 64] = acc[e >> 4][e & 15];
}
template <class G, int N>
__device__ __forceinline__ void sum_store(const float* x, int rg, int s, int lane, float scale, bf16_t* dst, bool on) {
  const int hh = lane >> 5;
#pragma unroll
  for (int c = 0; c < G::OWN / 4; ++c) {
    bf16x4 o;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      float v = 0.f;
#pragma unroll
      for (int p = 0; p < N; ++p) v += x[((size_t)(p * G::RG + rg) * G::NS + s * G::OWN + 4 * c + e) * 64 + lane];
      o[e] = (bf16_t)(scale * v);
    }
    // slot e holds d = 8 (e / 4) + 4 hh + e%4
    if (on) *(bf16x4*)(dst + 8 * (s * (G::OWN / 4) + c) + 4 * hh) = o;
  }
}

// ---------------------------------------------------------------- query-tile pass

template <int D, int KS>
__global__ __launch_bounds__(NTHREADS) __attribute__((amdgpu_waves_per_eu(2, 2)))
void attn_bwd_dq_split_kernel(const BwdArgs a) {
  using G = SGeo<D, KS>;
  constexpr int TB = G::TILEB, STB = 2 * KS * TB, VB = KS * TB;  // stage: K tiles, V tiles
  __shared__ __attribute__((aligned(1024))) char lds[2 * STB > G::XCHG ? 2 * STB : G::XCHG];

  const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
  const int lane = threadIdx.x & 63;
  const int hh = lane >> 5;
  const int rg = wave % G::RG, ks = wave / G::RG;
  const int L = a.L;

  const TileSlot sl = slot_of(blockIdx.x, a.B * a.H, a.order.nt, kHeadGroup);
  const int bh = sl.bh;
  int q0, q1;  // (the tile may be cut at a group bound: its rows end at q1)
  tile_rows(a.order, tile_of(a.order, sl.pos), G::BR, L, &q0, &q1);
  const size_t head = (size_t)bh * L * D;
  const bf16_t* __restrict__ Qg = (const bf16_t*)a.Q + head;
  const bf16_t* __restrict__ Kg = (const bf16_t*)a.K + head;
  const bf16_t* __restrict__ Vg = (const bf16_t*)a.V + head;
  const bf16_t* __restrict__ Og = (const bf16_t*)a.O + head;
  const bf16_t* __restrict__ gOg = (const bf16_t*)a.gO + head;
  const TilePlan plan = plan_tile(a.gt, q0, q1, BC);
  const int nblk = plan_num_blocks(plan);
  const int niter = (nblk + KS - 1) / KS;

  const unsigned lds0 = __builtin_amdgcn_readfirstlane(lds_addr(lds));
  const unsigned own = lds0 + (unsigned)(ks * TB);
  auto load = [&](int i, unsigned st) {  // the split's waves share its block's loads
    if (i >= nblk) return;
    const int k0 = plan_block(plan, i) * BC;
    load_rows<D, G::IPW>(Kg, k0, L, rg * G::IPW, own + st, lane);
    load_rows<D, G::IPW>(Vg, k0, L, rg * G::IPW, own + st + VB, lane);
  };
  load(ks, 0);

  const int row = q0 + rg * 32 + (lane & 31);
  const int wrow0 = imin(q0 + rg * 32, q1 - 1);
  const WaveRanges wr = wave_ranges(a.gt, wrow0, imin(wrow0 + 31, q1 - 1));
  // Q^T and gO^T as B operands (lane: row l%32, d = 16 s + 8 (l/32) + 0..7), Delta of the row
  const size_t rbase = (size_t)imin(row, L - 1) * D;
  bf16x8 qop[G::KSTEPS], gop[G::KSTEPS];
  float dpart = 0.f;
#pragma unroll
  for (int s = 0; s < G::KSTEPS; ++s) {
    qop[s] = *(const bf16x8*)(Qg + rbase + 16 * s + 8 * hh);
    gop[s] = *(const bf16x8*)(gOg + rbase + 16 * s + 8 * hh);
    const bf16x8 ov = *(const bf16x8*)(Og + rbase + 16 * s + 8 * hh);
#pragma unroll
    for (int j = 0; j < 8; ++j) dpart = fmaf((float)gop[s][j], (float)ov[j], dpart);
  }
  const float delta = dpart + xor32(dpart);
  f32x16 ndelta;  // the gP sums start from -Delta
#pragma unroll
  for (int e = 0; e < 16; ++e) ndelta[e] = -delta;
  asm volatile("" : "+v"(ndelta));  // (held in registers, not formed again for each block)
  const float lse = a.LSE[(size_t)bh * L + imin(row, L - 1)];
  const float lse2 = lse == -INFINITY ? 0.f : lse * kLog2e;  // (a row without keys: all masked)
  if (row < q1 && hh == 0 && ks == 0) a.Delta[(size_t)bh * L + row] = delta;

  unsigned trx[2];
  tr_bases<D>(lane, trx);
  const unsigned koff = lds_off<D>(lane & 31, hh);
  f32x16 gacc[G::DT];
#pragma unroll
  for (int dt = 0; dt < G::DT; ++dt) gacc[dt] = f32x16{};
  const float c2 = a.scale * kLog2e;

  __builtin_amdgcn_s_waitcnt(0xF70);  // (builtin: also retires the operand loads above)
  sync_all();
  for (int j = 0; j < niter; ++j) {
    const int i = j * KS + ks;
    const unsigned cur = (unsigned)((j & 1) * STB);
    load(i + KS, (unsigned)STB - cur);
    bool active = i < nblk;
    BlockMask mask{};
    if (active) {
      mask = block_mask(a.gt, wr, plan, row, plan_block(plan, i) * BC, L);
      active = !mask.none;
    }
    if (active) {
      // S^T = K Q^T and gP^T = V gO^T, operands read SPF k steps ahead
      f32x16 S = f32x16{}, GP = ndelta;
      const unsigned kb = vreg_add(own + cur, koff, j);
      constexpr int SPF = 2;
      bf16x8 kop[SPF + 1], vop[SPF + 1];
      auto read = [&](int s) {
        kop[s % (SPF + 1)] = ld128_at(kb ^ (32u * s));
        vop[s % (SPF + 1)] = ld128_at((kb ^ (32u * s)) + VB);
      };
#pragma unroll
      for (int s = 0; s < SPF; ++s) read(s);
#pragma unroll
      for (int s = 0; s < G::KSTEPS; ++s) {
        if (s + SPF < G::KSTEPS) read(s + SPF);
        __builtin_amdgcn_sched_barrier(0);
        S = mfma(kop[s % (SPF + 1)], qop[s], S);
        GP = mfma(vop[s % (SPF + 1)], gop[s], GP);
        __builtin_amdgcn_sched_barrier(0);
      }
      // P^T = exp(S^T - LSE) on admissible pairs, gS^T = P^T o (gP^T - Delta)
      float p[16];
#pragma unroll
      for (int e = 0; e < 16; ++e) p[e] = __builtin_amdgcn_exp2f(fmaf(S[e], c2, -lse2));
      if (!mask.all) {
        const uint32_t bits = mask.bits >> (4 * hh);
#pragma unroll
        for (int e = 0; e < 16; ++e) p[e] = ((bits >> (8 * (e >> 2) + (e & 3))) & 1u) ? p[e] : 0.f;
      }
      bf16x8 gsb[2];
#pragma unroll
      for (int e = 0; e < 16; ++e) gsb[e >> 3][e & 7] = (bf16_t)(p[e] * GP[e]);
      // gQ^T += K^T gS^T
      const unsigned tb0 = vreg_add(own + cur, trx[0], j), tb1 = vreg_add(own + cur, trx[1], j);
      constexpr int OPF = 2, NG = 2 * G::DT;
      bf16x8 kt[OPF + 1];
      auto read_t = [&](int g) {
        const int t = g / G::DT, dt = g % G::DT;
        const unsigned o = 16u * t * G::ROWB;
        kt[g % (OPF + 1)] = cat(ld_tr_at((tb0 ^ (64u * dt)) + o), ld_tr_at((tb1 ^ (64u * dt)) + o));
      };
#pragma unroll
      for (int g = 0; g < OPF; ++g) read_t(g);
#pragma unroll
      for (int g = 0; g < NG; ++g) {
        if (g + OPF < NG) read_t(g + OPF);
        __builtin_amdgcn_sched_barrier(0);
        gacc[g % G::DT] = mfma(kt[g % (OPF + 1)], gsb[g / G::DT], gacc[g % G::DT]);
        __builtin_amdgcn_sched_barrier(0);
      }
    }
    sync_all();  // round j is done with its stage, the loads of round j + 1 have landed
  }

  put<G, KS>((float*)lds, wave, lane, gacc);
  __syncthreads();
  sum_store<G, KS>((const float*)lds, rg, ks, lane, a.scale, (bf16_t*)a.gQ + head + (size_t)row * D, row < q1);
}

// ---------------------------------------------------------------- key-tile pass

template <int D, int RS>
__global__ __launch_bounds__(NTHREADS) __attribute__((amdgpu_waves_per_eu(2, 2)))
void attn_bwd_dkdv_split_kernel(const BwdArgs a) {
  using G = SGeo<D, RS>;
  // a stage holds, per split, the Q and gO tiles of a 32-row block and its LSE and Delta (64
  // values each are loaded, 32 are read); then the V tile, and the keys' query intervals
  constexpr bool NEGV = kNegV<D>;  // V is held negated, and the sums Delta - gO V^T start from Delta
  constexpr int TB = G::TILEB, STB = 2 * RS * TB + RS * 512, GB = RS * TB, SB = 2 * RS * TB;
  constexpr int VT = 2 * STB, WT = VT + G::BR * G::ROWB, BYTES = WT + 16 * G::BR;
  static_assert(STB % 1024 == 0 && VT % 1024 == 0, "XOR-formed offsets need row-aligned tiles");
  static_assert(G::RG >= 2, "two waves of a split load its row statistics");
  __shared__ __attribute__((aligned(1024))) char lds[BYTES > G::XCHG ? BYTES : G::XCHG];

  const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
  const int lane = threadIdx.x & 63;
  const int hh = lane >> 5;
  const int kg = wave % G::RG, rs = wave / G::RG;
  const int L = a.L;

  const TileSlot sl = slot_of(blockIdx.x, a.B * a.H, a.order.nt, kHeadGroupWide);
  const int bh = sl.bh;
  int k0, k1;
  tile_rows(a.order, tile_of(a.order, sl.pos), G::BR, L, &k0, &k1);
  const size_t head = (size_t)bh * L * D;
  const bf16_t* __restrict__ Qg = (const bf16_t*)a.Q + head;
  const bf16_t* __restrict__ Kg = (const bf16_t*)a.K + head;
  const bf16_t* __restrict__ Vg = (const bf16_t*)a.V + head;
  const bf16_t* __restrict__ gOg = (const bf16_t*)a.gO + head;
  const float* __restrict__ LSEg = a.LSE + (size_t)bh * L;
  const float* __restrict__ Dg = a.Delta + (size_t)bh * L;

  const GroupBits gbits = key_tile_bits(a.gt, k0, k1, lane);
  const TilePlan plan = plan_key_groups(a.gt, gbits, BC);
  const int nblk = plan_num_blocks(plan);
  const int niter = (nblk + RS - 1) / RS;

  const unsigned lds0 = __builtin_amdgcn_readfirstlane(lds_addr(lds));
  const unsigned own = lds0 + (unsigned)(rs * TB);
  const unsigned stat = lds0 + (unsigned)(SB + rs * 512);
  auto load = [&](int i, unsigned st) {
    if (i >= nblk) return;
    const int r0 = plan_block(plan, i) * BC;
    load_rows<D, G::IPW>(Qg, r0, L, kg * G::IPW, own + st, lane);
    load_rows<D, G::IPW>(gOg, r0, L, kg * G::IPW, own + st + GB, lane);
    const unsigned roff = (unsigned)imin(r0 + lane, L - 1) * 4u;
    if (kg == 0) lds_load4(LSEg, roff, stat + st);
    if (kg == 1) lds_load4(Dg, roff, stat + st + 256);
  };
  load(rs, 0);
  // the V tile (IPT loads per 32 keys), and the K operands of this wave's keys in registers
#pragma unroll
  for (int j0 = 0; j0 < G::RG * G::IPT; j0 += NW)
    if ((G::RG * G::IPT) % NW == 0 || j0 + wave < G::RG * G::IPT)
      load_rows<D, 1>(Vg, k0, L, j0 + wave, lds0 + VT, lane);
  const int krow = kg * 32 + (lane & 31);
  const int key = k0 + krow;
  bf16x8 kreg[G::KSTEPS];
#pragma unroll
  for (int s = 0; s < G::KSTEPS; ++s) kreg[s] = *(const bf16x8*)(Kg + (size_t)imin(key, L - 1) * D + 16 * s + 8 * hh);
  const int4* const windows = (const int4*)(lds + WT);
  const bool direct = key_window_table(a.gt, gbits, k0, G::BR, k1, (int4*)(lds + WT));

  unsigned trx[2];
  tr_bases<D>(lane, trx);
  const unsigned qoff = lds_off<D>(lane & 31, hh);
  const unsigned voff = (unsigned)VT + lds_off<D>(krow, hh);
  f32x16 gk[G::DT], gv[G::DT];
#pragma unroll
  for (int dt = 0; dt < G::DT; ++dt) {
    gk[dt] = f32x16{};
    gv[dt] = f32x16{};
  }
  const float c2 = a.scale * kLog2e;

  __builtin_amdgcn_s_waitcnt(0xF70);
  if constexpr (NEGV) {  // (each lane flips the pieces that it loaded itself)
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
#pragma unroll
    for (int j0 = 0; j0 < G::RG * G::IPT; j0 += NW)
      if ((G::RG * G::IPT) % NW == 0 || j0 + wave < G::RG * G::IPT)
        flip_signs(lds0 + (unsigned)(VT + (j0 + wave) * 1024 + lane * 16));
  }
  sync_all();
  for (int j = 0; j < niter; ++j) {
    const int i = j * RS + rs;
    const unsigned cur = (unsigned)((j & 1) * STB);
    load(i + RS, (unsigned)STB - cur);
    bool active = i < nblk, full = true;
    uint32_t bits = ~0u;
    if (active) {
      const int qw = plan_block(plan, i) * BC;
      full = block_is_full(plan, qw, BC, L);
      if (!full) {
        bits = direct ? window_bits(windows[krow], qw) : key_bits(a.gt, key, qw, L);
        active = __ballot(bits != 0) != 0;
      }
    }
    if (active) {
      // S = Q K^T and gP = gO V^T (lane: key l%32, rows 8 (i/4) + 4 (l/32) + i%4), operands
      // read one k step ahead
      f32x16 S = f32x16{}, GP = f32x16{};
      const float* const sl4 = (const float*)(lds + SB + rs * 512 + cur);
      if constexpr (NEGV) GP = acc_rows(sl4 + 64 + 4 * hh);
      const unsigned qa = vreg_add(own + cur, qoff, j), vb = vreg_add(lds0, voff, j);
      bf16x8 aq[2], ag[2], bv[2];
      auto read = [&](int s) {
        aq[s & 1] = ld128_at(qa ^ (32u * s));
        ag[s & 1] = ld128_at((qa ^ (32u * s)) + GB);
        bv[s & 1] = ld128_at(vb ^ (32u * s));
      };
      read(0);
#pragma unroll
      for (int s = 0; s < G::KSTEPS; ++s) {
        if (s + 1 < G::KSTEPS) read(s + 1);
        __builtin_amdgcn_sched_barrier(0);
        S = mfma(aq[s & 1], kreg[s], S);
        GP = mfma(ag[s & 1], bv[s & 1], GP);
        __builtin_amdgcn_sched_barrier(0);
      }
      // a row without admissible keys has LSE = -inf: exp2 then gives +inf, which the mask
      // (such a row is never in a full block) replaces by 0
      float p[16];
      bf16x8 pb[2], gsb[2];
#pragma unroll
      for (int c = 0; c < 4; ++c) {
        const float4 lv = *(const float4*)(sl4 + 8 * c + 4 * hh);
        const float lsev[4] = {lv.x, lv.y, lv.z, lv.w};
#pragma unroll
        for (int e = 0; e < 4; ++e) p[4 * c + e] = __builtin_amdgcn_exp2f(fmaf(S[4 * c + e], c2, -lsev[e] * kLog2e));
      }
      if (!full) {
        const uint32_t b = bits >> (4 * hh);
#pragma unroll
        for (int e = 0; e < 16; ++e) p[e] = ((b >> (8 * (e >> 2) + (e & 3))) & 1u) ? p[e] : 0.f;
      }
#pragma unroll
      for (int c = 0; c < 4; ++c) {
        const float4 dv = NEGV ? float4{} : *(const float4*)(sl4 + 64 + 8 * c + 4 * hh);
        const float dlv[4] = {dv.x, dv.y, dv.z, dv.w};
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const int x = 4 * c + e;
          pb[x >> 3][x & 7] = (bf16_t)p[x];
          gsb[x >> 3][x & 7] = (bf16_t)(NEGV ? p[x] * GP[x] : p[x] * (GP[x] - dlv[e]));  // (NEGV: -gS)
        }
      }
      // gV^T += gO^T P and gK^T += Q^T gS
      constexpr int NG = 2 * G::DT;
      const unsigned tb0 = vreg_add(own + cur, trx[0], j), tb1 = vreg_add(own + cur, trx[1], j);
      bf16x8 got[2], qt[2];
      auto read_t = [&](int g) {
        const int t = g / G::DT, dt = g % G::DT;
        const unsigned o = 16u * t * G::ROWB;
        const unsigned a0 = (tb0 ^ (64u * dt)) + o, a1 = (tb1 ^ (64u * dt)) + o;
        got[g & 1] = cat(ld_tr_at(a0 + GB), ld_tr_at(a1 + GB));
        qt[g & 1] = cat(ld_tr_at(a0), ld_tr_at(a1));
      };
      read_t(0);
#pragma unroll
      for (int g = 0; g < NG; ++g) {
        if (g + 1 < NG) read_t(g + 1);
        __builtin_amdgcn_sched_barrier(0);
        const int t = g / G::DT, dt = g % G::DT;
        gv[dt] = mfma(got[g & 1], pb[t], gv[dt]);
        gk[dt] = mfma(qt[g & 1], gsb[t], gk[dt]);
        __builtin_amdgcn_sched_barrier(0);
      }
    }
    sync_all();
  }

  float* const x = (float*)lds;
  put<G, RS>(x, wave, lane, gk);
  __syncthreads();
  sum_store<G, RS>(x, kg, rs, lane, NEGV ? -a.scale : a.scale, (bf16_t*)a.gK + head + (size_t)key * D, key < k1);
  __syncthreads();
  put<G, RS>(x, wave, lane, gv);
  __syncthreads();
  sum_store<G, RS>(x, kg, rs, lane, 1.f, (bf16_t*)a.gV + head + (size_t)key * D, key < k1);
}

}  // namespace

void launch_bwd_dq_split(const BwdArgs& a, int D, hipStream_t stream) {
  const dim3 grid((unsigned)(a.order.nt * a.B * a.H)), block(NTHREADS);
  if (D == 128) {
    if (a.split == 4) hipLaunchKernelGGL((attn_bwd_dq_split_kernel<128, 4>), grid, block, 0, stream, a);
    else hipLaunchKernelGGL((attn_bwd_dq_split_kernel<128, 2>), grid, block, 0, stream, a);
  } else {
    if (a.split == 4) hipLaunchKernelGGL((attn_bwd_dq_split_kernel<64, 4>), grid, block, 0, stream, a);
    else hipLaunchKernelGGL((attn_bwd_dq_split_kernel<64, 2>), grid, block, 0, stream, a);
  }
}

void launch_bwd_dkdv_split(const BwdArgs& a, int D, hipStream_t stream) {
  const dim3 grid((unsigned)(a.order.nt * a.B * a.H)), block(NTHREADS);
  if (D == 128) hipLaunchKernelGGL((attn_bwd_dkdv_split_kernel<128, 4>), grid, block, 0, stream, a);
  else hipLaunchKernelGGL((attn_bwd_dkdv_split_kernel<64, 4>), grid, block, 0, stream, a);
}

}  // namespace attn
