// Block-causal attention backward (gfx950): the analytic softmax gradient of
// paper Sec. 3.2's attention, with P recomputed from Q, K and the forward LSE.
//
//   row-term kernel : Delta_i = sum_d dO_id O_id                 (HBM-bound)
//   one grid of two kinds of workgroups:
//   dK/dV work : a workgroup owns 128 or 64 keys (32 per wave, K held in
//                registers, V in registers or, at D = 128, mostly in LDS); it
//                walks the query tiles that can see those keys -- queries of the same or
//                a later chunk -- staging Q, dO, LSE and Delta in LDS.  Per 32
//                queries and wave:
//                  S = Q K^T, dP = dO V^T     (keys on the lane axis)
//                  P = exp(S - LSE), dS = P (dP - Delta)
//                  dV^T += dO^T P, dK^T += Q^T dS   (transposing LDS reads)
//   dQ work    : a workgroup owns 128 or 64 queries (Q and dO in registers) and
//                walks the key tiles below the chunk diagonal:
//                  S^T = K Q^T, dP^T = V dO^T, dS^T = P^T (dP^T - Delta)
//                  dQ^T += K^T dS^T
// Recomputing S and dP in the dQ work costs 1.4x the MFMA work of a fused
// kernel with atomic dQ updates, but needs no fp32 dQ buffer and gives a
// deterministic result.
#include <type_traits>

#include "mw_device.h"
#include "mw_kernels.h"

namespace mw {

// Row terms of the backward pass: -Delta = -rowsum(dO * O) and LSE scaled to
// base 2 (LSE * log2 e), one 16-byte chunk per thread, reduced over the row's
// lanes.  Delta is stored negated: the dP products start from it (their MFMA
// accumulator input), so dP - Delta costs no instruction.
// CPR lanes per row (a power of two); at D = 72 the 9 pieces of a row leave
// lanes 9..15 of its group idle.
template <int D>
__global__ __launch_bounds__(256) void bwd_rowterms_kernel(BwdParams p, long long n_rows) {
  constexpr int CPR = D == 64 ? 8 : 16;
  const long long gid = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  const long long row = gid / CPR;
  const int c = (int)(gid % CPR);
  float acc = 0.f;
  if (row < n_rows && c < D / 8) {
    const long long bh = row / p.T, t = row - bh * p.T, bi = bh / p.H, hi = bh - bi * p.H;
    const u32x4 a = *reinterpret_cast<const u32x4*>(p.o + bi * p.so.b + hi * p.so.h + t * p.so.t + c * 8);
    const u32x4 b = *reinterpret_cast<const u32x4*>(p.d_o + bi * p.sdo.b + hi * p.sdo.h + t * p.sdo.t + c * 8);
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const float a0 = __uint_as_float(a[j] << 16), a1 = __uint_as_float(a[j] & 0xffff0000u);
      const float b0 = __uint_as_float(b[j] << 16), b1 = __uint_as_float(b[j] & 0xffff0000u);
      acc = fmaf(a0, b0, acc);
      acc = fmaf(a1, b1, acc);
    }
  }
#pragma unroll
  for (int w = CPR / 2; w >= 1; w >>= 1) acc += __shfl_xor(acc, w);
  if (row < n_rows && c == 0) {
    p.delta[row] = -acc;
    p.lse2[row] = p.lse[row] * 1.4426950408889634f;
  }
}

// LDS of the dK/dV work: Q and dO tiles of BS queries (two stages each), then LSE
// and -Delta of the tile's rows (two stages each, staged 64 rows at a time), then
// VL V fragments of each key wave (see dkdv_body).
template <int D, int NW, int QG, int BM, int VL>
struct DkdvLds {
  static constexpr int BS = BM * QG;
  static constexpr int TE = stage_elems<D, BS, 64 * NW>();
  static constexpr int RT = BS < 64 ? 64 : BS;  // row-term entries per stage
  static constexpr int BYTES = 2 * 2 * TE * 2 + 2 * 2 * RT * 4 + (NW / QG) * VL * 1024;
};

// Sum of the partial accumulators of G wave groups into group 0, through LDS:
// in each round the upper half of the remaining groups hands its tiles to the
// lower half (a fixed order, so the result is deterministic).  `slot` is the
// wave's index in its group of NWG waves; every wave of the workgroup calls it
// after the last read of `lds`.
template <int G, int NWG, int NA>
__device__ __forceinline__ void merge_groups(f32x16 (&acc)[NA], const int group, const int slot, const int lane,
                                             unsigned char* lds) {
  float* x = reinterpret_cast<float*>(lds);
#pragma unroll
  for (int half = G / 2; half >= 1; half >>= 1) {
    if (half != G / 2) __syncthreads();  // the previous round has been read
    const int at = ((group - half) * NWG + slot) * NA;
    if (group >= half && group < 2 * half) {
#pragma unroll
      for (int n = 0; n < NA; ++n)
#pragma unroll
        for (int i = 0; i < 16; ++i) x[((at + n) * 16 + i) * 64 + lane] = acc[n][i];
    }
    __syncthreads();
    if (group < half) {
      const int from = (group * NWG + slot) * NA;
#pragma unroll
      for (int n = 0; n < NA; ++n)
#pragma unroll
        for (int i = 0; i < 16; ++i) acc[n][i] += x[((from + n) * 16 + i) * 64 + lane];
    }
  }
}
template <int G, int NWG, int NA>
constexpr int merge_bytes() {
  return G == 1 ? 0 : (G / 2) * NWG * NA * 16 * 64 * 4;
}

// NW waves in QG query groups of NW / QG key waves.  A wave owns 32 keys (K and
// V fragments and the dK, dV accumulators in registers); a step stages BM * QG
// queries, of which a group takes its BM, and the groups' dK and dV are summed
// through LDS at the end: QG groups walk a key tile's queries in 1 / QG of the
// steps, for grids too small to fill the card with whole chains.  The first VL
// V fragments (the dP products' B operand) are read from LDS, where they are
// staged once as they lie in the registers (fragment kk of key wave kw: 16
// bytes per lane), so a read needs no swizzle and one address for all: 4 VL
// registers fewer per wave for VL more 1 KB reads per 32 x 32 block.  Work item:
// key tile kt of (batch, head) bh.
template <int D, int NW, int QG, int BM, int VL>
__device__ __forceinline__ void dkdv_body(const BwdParams& p, const int bh, const int kt, unsigned char* lds) {
  static_assert(NW % QG == 0, "waves split evenly into query groups");
  constexpr int NWK = NW / QG, BN = 32 * NWK, NT = 64 * NW;
  static_assert(BM % 32 == 0, "32-row query blocks");
  constexpr int KK = (D + 15) / 16, DB = D / 32;  // D = 72: 80 columns, and a tail of 8 (Tail72)
  static_assert(16 * VL <= D, "the V fragments in LDS have no zero columns past D");
  using LD = DkdvLds<D, NW, QG, BM, VL>;
  constexpr int TE = LD::TE, RT = LD::RT, BS = LD::BS;
  bf16_t(*Qs)[TE] = reinterpret_cast<bf16_t(*)[TE]>(lds);
  bf16_t(*dOs)[TE] = reinterpret_cast<bf16_t(*)[TE]>(lds + 2 * TE * 2);
  float(*lse_s)[RT] = reinterpret_cast<float(*)[RT]>(lds + 4 * TE * 2);
  float(*dlt_s)[RT] = reinterpret_cast<float(*)[RT]>(lds + 4 * TE * 2 + 2 * RT * 4);
  bf16_t* Vs = reinterpret_cast<bf16_t*>(lds + 4 * TE * 2 + 4 * RT * 4);  // V fragments [key wave][VL][64 lanes][8]

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = QG == 1 ? tid >> 6 : __builtin_amdgcn_readfirstlane(tid >> 6);
  const int kw = QG == 1 ? wave : wave % NWK, qg = QG == 1 ? 0 : wave / NWK;  // key wave, query group
  const int gq = qg * BM;                 // the group's first row of a staged tile
  const FragOffsets<D> fo(lane, gq * D);  // Q and dO tiles share the layout
  const bf16_t* vfrag = Vs + (kw * VL * 64 + lane) * 8;
  const int T = p.T, L = p.L;
  const int k0 = kt * BN;
  const int bi = bh / p.H, hi = bh - bi * p.H;
  const long long qb_ = bi * p.sq.b + hi * p.sq.h, dob_ = bi * p.sdo.b + hi * p.sdo.h;
  const float* lse2_bh = p.lse2 + (long long)bh * T;
  const float* dlt_bh = p.delta + (long long)bh * T;

  // This lane's key, the first query that sees it, and its K and V fragments (B
  // operands of S = Q K^T and dP = dO V^T).  Keys past T read the last key;
  // their dK/dV are never stored.
  const int mykey = k0 + kw * 32 + (lane & 31);
  const long long kr = min(mykey, T - 1);
  const int qvis = ((int)kr / L) * L;
  bf16x8 kf[KK], vf[KK];
  const bf16_t* ka = p.k + bi * p.sk.b + hi * p.sk.h + kr * p.sk.t + 8 * (lane >> 5);
  const bf16_t* va = p.v + bi * p.sv.b + hi * p.sv.h + kr * p.sv.t + 8 * (lane >> 5);
#pragma unroll
  for (int kk = 0; kk < KK; ++kk) {
    if (D % 16 == 0 || 16 * kk + 8 * (lane >> 5) < D) {
      kf[kk] = *reinterpret_cast<const bf16x8*>(ka + 16 * kk);
      if (kk >= VL) vf[kk] = *reinterpret_cast<const bf16x8*>(va + 16 * kk);
    } else {  // columns past D (D = 72): zeros
#pragma unroll
      for (int j = 0; j < 8; ++j) kf[kk][j] = vf[kk][j] = (__bf16)0.f;
    }
  }
  constexpr bool TAIL = D % 32 != 0;
  const Tail72 ft(lane, gq * D);  // (TAIL)
  f32x4 tail[4] = {zero4(), zero4(), zero4(), zero4()};  // (TAIL) dV^T of keys 0..15 and 16..31, dK^T of the same
  f32x16 dv[DB], dk[DB];
#pragma unroll
  for (int db = 0; db < DB; ++db) {
    dv[db] = zero16();
    dk[db] = zero16();
  }

  const int klast = min(k0 + BN, T) - 1;
  const int qstart = ((k0 / L) * L / BS) * BS;  // first query tile with a query of chunk >= chunk(k0)
  const float c = p.scale_log2;

  const RowOffsets<D, BS, NT> ro_q(p.sq.t, tid), ro_do(p.sdo.t, tid);
  auto stage = [&](int q0, int b) {
    if (q0 + BS <= T) {  // whole tile: scalar base + per-thread offsets
      stage_rows_s<D, BS, NT>(Qs[b], p.q + qb_ + q0 * p.sq.t, ro_q, tid);
      stage_rows_s<D, BS, NT>(dOs[b], p.d_o + dob_ + q0 * p.sdo.t, ro_do, tid);
    } else {  // the ragged last tile: rows past T read the last row
      stage_rows_direct<D, BS, NT>(Qs[b], [&](int r) { return p.q + qb_ + min(q0 + r, T - 1) * p.sq.t; }, tid);
      stage_rows_direct<D, BS, NT>(dOs[b], [&](int r) { return p.d_o + dob_ + min(q0 + r, T - 1) * p.sdo.t; }, tid);
    }
    // row terms of the tile: 64 fp32 per wave, LSE then -Delta
#pragma unroll
    for (int c = wave; c < 2 * (RT / 64); c += NW) {
      const int part = c % (RT / 64);
      if (c < RT / 64) {
        stage_f32x64_direct(lse_s[b] + 64 * part, lse2_bh, q0 + 64 * part, T, lane);
      } else {
        stage_f32x64_direct(dlt_s[b] + 64 * part, dlt_bh, q0 + 64 * part, T, lane);
      }
    }
  };

  auto step = [&](auto masked, const int q0, const int buf) {
    const bf16_t* Qt = Qs[buf];
    const bf16_t* dOt = dOs[buf];
#pragma unroll
    for (int qb = 0; qb < BM / 32; ++qb) {
      // -Delta of the tile's rows in accumulator layout (register i: row
      // 8(i/4) + 4(l/32) + i%4): the dP products accumulate onto it
      f32x16 ndl;
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        const f32x4 d4 = *reinterpret_cast<const f32x4*>(&dlt_s[buf][gq + qb * 32 + 8 * g + 4 * (lane >> 5)]);
#pragma unroll
        for (int j = 0; j < 4; ++j) ndl[4 * g + j] = d4[j];
      }
      f32x16 s, dp;
      s = zero16();
      dp = ndl;
#pragma unroll
      for (int kk = 0; kk < KK; ++kk) {
        const bf16x8 qa = fo.row8(Qt, qb * 32, kk);
        const bf16x8 da = fo.row8(dOt, qb * 32, kk);
        s = mfma32(qa, kf[kk], s);
        const bf16x8 vk = kk < VL ? *reinterpret_cast<const bf16x8*>(vfrag + kk * 512) : vf[kk];
        dp = mfma32(da, vk, dp);
      }
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        const int rr = gq + qb * 32 + 8 * g + 4 * (lane >> 5);
        const f32x4 l4 = *reinterpret_cast<const f32x4*>(&lse_s[buf][rr]);
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          const int i = 4 * g + j;
          float pv = fast_exp2(fmaf(s[i], c, -l4[j]));
          if constexpr (decltype(masked)::value) {
            const int q = q0 + rr + j;
            const bool ok = (q < T) & (q >= qvis);  // q in the key's chunk or a later one
            pv = ok ? pv : 0.f;
          }
          s[i] = pv;
          dp[i] = pv * dp[i];  // P (dP - Delta)
        }
      }
      if constexpr (TAIL) {
        // P, then dS: only one's packed halves are alive at a time.  With both kept for
        // the tail the 128-row tile spilled seven registers around its loops, now one:
        // 16 heads x 19200 2914 -> 2890 us, 15 x 2999 97.7 -> 95.1
        bf16x8 h[2] = {pack8(s, 0), pack8(s, 1)};
#pragma unroll
        for (int t = 0; t < 2; ++t)
#pragma unroll
          for (int db = 0; db < DB; ++db) dv[db] = mfma32(fo.tr8(dOt, qb * 32, t, db), h[t], dv[db]);
        tail_operands(h[0], h[1]);
        const bf16x8 dot = ft.read(dOt, qb * 32);
#pragma unroll
        for (int e = 0; e < 2; ++e) tail[e] = mfma16(dot, h[e], tail[e]);
#pragma unroll
        for (int t = 0; t < 2; ++t) {
          h[t] = pack8(dp, t);
#pragma unroll
          for (int db = 0; db < DB; ++db) dk[db] = mfma32(fo.tr8(Qt, qb * 32, t, db), h[t], dk[db]);
        }
        tail_operands(h[0], h[1]);
        const bf16x8 qt = ft.read(Qt, qb * 32);
#pragma unroll
        for (int e = 0; e < 2; ++e) tail[2 + e] = mfma16(qt, h[e], tail[2 + e]);
      } else {
#pragma unroll
        for (int t = 0; t < 2; ++t) {
          const bf16x8 pb = pack8(s, t), dsb = pack8(dp, t);
#pragma unroll
          for (int db = 0; db < DB; ++db) {
            dv[db] = mfma32(fo.tr8(dOt, qb * 32, t, db), pb, dv[db]);
            dk[db] = mfma32(fo.tr8(Qt, qb * 32, t, db), dsb, dk[db]);
          }
        }
      }
    }
  };

  // Query tiles [qfb, qfe) see every key of this workgroup and are whole; the
  // ones before (same chunk as the keys) and the ragged last tile run masked.
  const int qfb = max(qstart, ((L * (klast / L) + BS - 1) / BS) * BS);
  const int qfe = max(qfb, (T / BS) * BS);
  int buf = 0;
  int q0 = qstart;
  for (int f = __builtin_amdgcn_readfirstlane(wave); f < NWK * VL; f += NW) {  // V fragments, one a wave and round
    const int w = f / (VL > 0 ? VL : 1), kk = f - w * VL;
    const long long row = min(k0 + w * 32 + (lane & 31), T - 1);
    dma_lds_16(p.v + bi * p.sv.b + hi * p.sv.h + row * p.sv.t + 16 * kk + 8 * (lane >> 5), lds_addr(Vs) + f * 1024);
  }
  if (q0 < T) stage(q0, 0);
  wait_vmem();
  __syncthreads();
  auto run = [&](auto masked, const int qstop) {
    for (; q0 < qstop; q0 += BS) {
      if (q0 + BS < T) stage(q0 + BS, buf ^ 1);  // next query tile streams in during this one
      step(masked, q0, buf);
      wait_vmem();
      __syncthreads();
      buf ^= 1;
    }
  };
  run(std::true_type{}, min(qfb, T));
  run(std::false_type{}, min(qfe, T));
  run(std::true_type{}, T);

  if constexpr (QG > 1) {
    merge_groups<QG, NWK>(dv, qg, kw, lane, lds);
    __syncthreads();
    merge_groups<QG, NWK>(dk, qg, kw, lane, lds);
    if constexpr (TAIL) {
      f32x16 all[1];
#pragma unroll
      for (int i = 0; i < 16; ++i) all[0][i] = tail[i / 4][i % 4];
      __syncthreads();
      merge_groups<QG, NWK>(all, qg, kw, lane, lds);
#pragma unroll
      for (int i = 0; i < 16; ++i) tail[i / 4][i % 4] = all[0][i];
    }
    if (qg > 0) return;  // no barrier follows
  }
  if constexpr (TAIL) {
    if (lane < 32) {  // columns 64 + 4 (l / 16) + i of keys l % 16 and 16 + l % 16
#pragma unroll
      for (int e = 0; e < 2; ++e) {
        const int key = k0 + kw * 32 + 16 * e + (lane & 15), col = 64 + 4 * (lane >> 4);
        if (key >= T) continue;
        bf16x4 wk, wv;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          wk[j] = to_bf16(tail[2 + e][j] * p.scale);
          wv[j] = to_bf16(tail[e][j]);
        }
        *reinterpret_cast<bf16x4*>(p.dk + bi * p.sdk.b + hi * p.sdk.h + key * p.sdk.t + col) = wk;
        *reinterpret_cast<bf16x4*>(p.dv + bi * p.sdv.b + hi * p.sdv.h + key * p.sdv.t + col) = wv;
      }
    }
  }
  if (mykey >= T) return;
  bf16_t* dkrow = p.dk + bi * p.sdk.b + hi * p.sdk.h + mykey * p.sdk.t;
  bf16_t* dvrow = p.dv + bi * p.sdv.b + hi * p.sdv.h + mykey * p.sdv.t;
#pragma unroll
  for (int db = 0; db < DB; ++db) {
#pragma unroll
    for (int g = 0; g < 4; ++g) {
      bf16x4 wk, wv;
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        wk[j] = to_bf16(dk[db][4 * g + j] * p.scale);
        wv[j] = to_bf16(dv[db][4 * g + j]);
      }
      const int col = db * 32 + 8 * g + 4 * (lane >> 5);
      *reinterpret_cast<bf16x4*>(dkrow + col) = wk;
      *reinterpret_cast<bf16x4*>(dvrow + col) = wv;
    }
  }
}

// LDS of the dQ work: K and V tiles of BS keys, two stages each.
template <int D, int NW, int BS>
struct DqLds {
  static constexpr int TE = stage_elems<D, BS, 64 * NW>();
  static constexpr int BYTES = 2 * 2 * TE * 2;
};

// NW waves in KG key groups of NW / KG row waves, each wave owning 32 query
// rows; a step stages BN * KG keys, of which a group takes its BN, and the
// groups' dQ are summed through LDS at the end.  Work item: query tile qt of
// (batch, head) bh.
template <int D, int NW, int KG, int BN>
__device__ __forceinline__ void dq_body(const BwdParams& p, const int bh, const int qt, unsigned char* lds) {
  static_assert(NW % KG == 0, "waves split evenly into key groups");
  constexpr int NWR = NW / KG, BM = 32 * NWR, NT = 64 * NW, BS = BN * KG;
  constexpr int KK = (D + 15) / 16, DB = D / 32;  // D = 72: 80 columns, and a tail of 8 (Tail72)
  constexpr int TE = DqLds<D, NW, BS>::TE;
  bf16_t(*Ks)[TE] = reinterpret_cast<bf16_t(*)[TE]>(lds);
  bf16_t(*Vs)[TE] = reinterpret_cast<bf16_t(*)[TE]>(lds + 2 * TE * 2);

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = KG == 1 ? tid >> 6 : __builtin_amdgcn_readfirstlane(tid >> 6);
  const int rw = KG == 1 ? wave : wave % NWR, kg = KG == 1 ? 0 : wave / NWR;  // row wave, key group
  const FragOffsets<D> fo(lane, kg * BN * D);  // K and V tiles share the layout
  const int T = p.T, L = p.L;
  const int q0 = qt * BM;
  const int bi = bh / p.H, hi = bh - bi * p.H;
  const long long kb_ = bi * p.sk.b + hi * p.sk.h, vb_ = bi * p.sv.b + hi * p.sv.h;

  const int qrow = q0 + rw * 32 + (lane & 31);
  const int qc = min(qrow, T - 1);
  bf16x8 qf[KK], df[KK];
  const bf16_t* qa = p.q + bi * p.sq.b + hi * p.sq.h + qc * p.sq.t + 8 * (lane >> 5);
  const bf16_t* da = p.d_o + bi * p.sdo.b + hi * p.sdo.h + qc * p.sdo.t + 8 * (lane >> 5);
#pragma unroll
  for (int kk = 0; kk < KK; ++kk) {
    if (D % 16 == 0 || 16 * kk + 8 * (lane >> 5) < D) {
      qf[kk] = *reinterpret_cast<const bf16x8*>(qa + 16 * kk);
      df[kk] = *reinterpret_cast<const bf16x8*>(da + 16 * kk);
    } else {  // columns past D (D = 72): zeros
#pragma unroll
      for (int j = 0; j < 8; ++j) qf[kk][j] = df[kk][j] = (__bf16)0.f;
    }
  }
  const float lse2 = p.lse2[(long long)bh * T + qc];  // LSE * log2 e and -Delta of this lane's query
  const float ndlt = p.delta[(long long)bh * T + qc];
  const int e1 = min(T, (qc / L + 1) * L);
  const int e1f = min(T, (q0 / L + 1) * L);
  const int kend = min(T, ((min(q0 + BM, T) - 1) / L + 1) * L);
  const float c = p.scale_log2;
  // -Delta depends only on the query (the lane's accumulator column): a tile
  // of it is the accumulator input of every dP product, so dS = P (dP - Delta)
  // is one multiply per element
  f32x16 ndl;
#pragma unroll
  for (int i = 0; i < 16; ++i) ndl[i] = ndlt;

  constexpr bool TAIL = D % 32 != 0;
  const Tail72 ft(lane, kg * BN * D);        // (TAIL)
  f32x4 tail[2] = {zero4(), zero4()};        // (TAIL) dQ^T of queries 0..15 and 16..31
  f32x16 dq[DB];
#pragma unroll
  for (int db = 0; db < DB; ++db) dq[db] = zero16();

  const RowOffsets<D, BS, NT> ro_k(p.sk.t, tid), ro_v(p.sv.t, tid);
  auto stage = [&](int k0, int b) {
    if (k0 + BS <= T) {  // whole tile: scalar base + per-thread offsets
      stage_rows_s<D, BS, NT>(Ks[b], p.k + kb_ + k0 * p.sk.t, ro_k, tid);
      stage_rows_s<D, BS, NT>(Vs[b], p.v + vb_ + k0 * p.sv.t, ro_v, tid);
    } else {  // the ragged last tile: rows past T read the last row
      stage_rows_direct<D, BS, NT>(Ks[b], [&](int r) { return p.k + kb_ + min(k0 + r, T - 1) * p.sk.t; }, tid);
      stage_rows_direct<D, BS, NT>(Vs[b], [&](int r) { return p.v + vb_ + min(k0 + r, T - 1) * p.sv.t; }, tid);
    }
  };
  auto step = [&](auto masked, const int k0, const int buf) {
    const bf16_t* Kt = Ks[buf];
    const bf16_t* Vt = Vs[buf];
#pragma unroll
    for (int kb = 0; kb < BN / 32; ++kb) {
      f32x16 s = zero16(), dp = ndl;
#pragma unroll
      for (int kk = 0; kk < KK; ++kk) {
        s = mfma32(fo.row8(Kt, kb * 32, kk), qf[kk], s);
        dp = mfma32(fo.row8(Vt, kb * 32, kk), df[kk], dp);
      }
#pragma unroll
      for (int i = 0; i < 16; ++i) {
        float pv = fast_exp2(fmaf(s[i], c, -lse2));
        if constexpr (decltype(masked)::value) {
          const int key = k0 + kg * BN + kb * 32 + acc_row(i, lane);
          pv = key < e1 ? pv : 0.f;
        }
        dp[i] = pv * dp[i];  // P (dP - Delta)
      }
      bf16x8 dsb[2];
#pragma unroll
      for (int t = 0; t < 2; ++t) {
        dsb[t] = pack8(dp, t);
#pragma unroll
        for (int db = 0; db < DB; ++db) dq[db] = mfma32(fo.tr8(Kt, kb * 32, t, db), dsb[t], dq[db]);
      }
      if constexpr (TAIL) {
        const bf16x8 ktr = ft.read(Kt, kb * 32);
        tail_operands(dsb[0], dsb[1]);
#pragma unroll
        for (int e = 0; e < 2; ++e) tail[e] = mfma16(ktr, dsb[e], tail[e]);
      }
    }
  };

  // key tiles [0, kfull) are visible to every query of the workgroup
  const int kfull = (e1f / BS) * BS;
  int buf = 0;
  int k0 = 0;
  stage(0, 0);
  wait_vmem();
  __syncthreads();
  auto run = [&](auto masked, const int kstop) {
    for (; k0 < kstop; k0 += BS) {
      if (k0 + BS < kend) stage(k0 + BS, buf ^ 1);
      step(masked, k0, buf);
      wait_vmem();
      __syncthreads();
      buf ^= 1;
    }
  };
  run(std::false_type{}, min(kfull, kend));
  run(std::true_type{}, kend);

  if constexpr (KG > 1) {
    merge_groups<KG, NWR>(dq, kg, rw, lane, lds);
    if constexpr (TAIL) {
      f32x16 all[1] = {zero16()};
#pragma unroll
      for (int i = 0; i < 8; ++i) all[0][i] = tail[i / 4][i % 4];
      __syncthreads();
      merge_groups<KG, NWR>(all, kg, rw, lane, lds);
#pragma unroll
      for (int i = 0; i < 8; ++i) tail[i / 4][i % 4] = all[0][i];
    }
    if (kg > 0) return;  // no barrier follows
  }
  if constexpr (TAIL) {
    if (lane < 32) {  // columns 64 + 4 (l / 16) + i of queries l % 16 and 16 + l % 16
#pragma unroll
      for (int e = 0; e < 2; ++e) {
        const int q = q0 + rw * 32 + 16 * e + (lane & 15);
        if (q >= T) continue;
        bf16x4 w;
#pragma unroll
        for (int j = 0; j < 4; ++j) w[j] = to_bf16(tail[e][j] * p.scale);
        *reinterpret_cast<bf16x4*>(p.dq + bi * p.sdq.b + hi * p.sdq.h + q * p.sdq.t + 64 + 4 * (lane >> 4)) = w;
      }
    }
  }
  if (qrow >= T) return;
  bf16_t* row = p.dq + bi * p.sdq.b + hi * p.sdq.h + qrow * p.sdq.t;
#pragma unroll
  for (int db = 0; db < DB; ++db) {
#pragma unroll
    for (int g = 0; g < 4; ++g) {
      const int col = db * 32 + 8 * g + 4 * (lane >> 5);
      bf16x4 w;
#pragma unroll
      for (int j = 0; j < 4; ++j) w[j] = to_bf16(dq[db][4 * g + j] * p.scale);
      *reinterpret_cast<bf16x4*>(row + col) = w;
    }
  }
}

// dK/dV and dQ work in one grid: the first n_dkdv workgroups take key tiles,
// the rest query tiles, so the query tiles fill the CUs that the key tiles' tail
// leaves idle and no kernel boundary separates them.  Each part keeps its own
// XCD-aware, heaviest-first order (tile_item).  Early keys are seen by the most
// queries and late queries see the most keys: both parts run their heaviest tiles
// first.
template <int D, int NW, int G, int BMK, int BNQ, int VL, int WPS>
__global__ __launch_bounds__(64 * NW, WPS) void bwd_grad_kernel(BwdParams p, int n_dkdv, int n_qtiles) {
  constexpr int B1 = DkdvLds<D, NW, G, BMK, VL>::BYTES, B2 = DqLds<D, NW, BNQ * G>::BYTES;
  constexpr int B3 = merge_bytes<G, NW / G, D / 32>();
  constexpr int B12 = B1 > B2 ? B1 : B2;
  __shared__ __attribute__((aligned(16))) unsigned char lds[B12 > B3 ? B12 : B3];
  const int id = blockIdx.x;
  int bh, r;
  if (id < n_dkdv) {
    tile_item(id, p.BH, bh, r);
    dkdv_body<D, NW, G, BMK, VL>(p, bh, r, lds);
  } else {
    tile_item(id - n_dkdv, p.BH, bh, r);
    dq_body<D, NW, G, BNQ>(p, bh, n_qtiles - 1 - r, lds);
  }
}

// Configurations of the gradient grid: NW waves in G query (dK/dV) or key (dQ)
// groups, BMK queries and BNQ keys per group and step, registers for WPS waves
// per SIMD.
template <int NW_, int G_, int BMK_, int BNQ_, int VL_, int WPS_>
struct BwdTile {
  static constexpr int NW = NW_, G = G_, BMK = BMK_, BNQ = BNQ_, VL = VL_, WPS = WPS_;
  static constexpr int ROWS = 32 * (NW / G);  // keys (dK/dV) and queries (dQ) per workgroup
};
// 128 keys or queries.  D = 128: V fragments in LDS and 32-query steps bring the
// dK/dV work under 256 registers (247), so it runs two waves per SIMD beside the
// dQ work in one grid; holding all of V in registers needed 448 registers, one
// wave per SIMD, in a grid of its own (the backward 5% slower, results
// bit-identical).  Two of the eight V fragments fit the registers that are left:
// 5% fewer LDS reads, 16 heads x 42240 23.25 -> 23.14 ms, x 9600 1272 -> 1264 us
// against all eight in LDS.
template <int D>
using Wide = BwdTile<4, 1, D == 128 ? 32 : 64, D == 64 ? 128 : 64, D == 128 ? 6 : 0, 2>;
// 128 keys or queries, D = 64: 64-key dQ steps halve the LDS, and 168 registers let
// three waves run per SIMD (one register is spilled around the loops, none in them).
using Wide3 = BwdTile<4, 1, 64, 64, 0, 3>;
// 64 keys or queries, two groups of two waves: half the chain.  (D = 128: with
// one V fragment in registers two workgroups fit a CU's LDS; with none, one.)
template <int D>
using Pairs = BwdTile<4, 2, 32, 32, D == 128 ? 7 : 0, 2>;
// 64 keys or queries, four groups of two waves: a quarter of the chain.
template <int D>
using Quads = BwdTile<8, 4, 32, 32, D == 128 ? 8 : 0, 2>;

template <int D, class C>
static hipError_t launch_grad(const BwdParams& p, hipStream_t stream) {
  const int n = (p.T + C::ROWS - 1) / C::ROWS;
  hipLaunchKernelGGL((bwd_grad_kernel<D, C::NW, C::G, C::BMK, C::BNQ, C::VL, C::WPS>), dim3(2 * n * p.BH), dim3(64 * C::NW),
                     0, stream, p, n * p.BH, n);
  return hipGetLastError();
}

template <int D>
static hipError_t launch_bwd_d(const BwdParams& p, hipStream_t stream) {
  const long long rows = (long long)p.BH * p.T;
  const long long threads = rows * (D == 64 ? 8 : 16);
  hipLaunchKernelGGL(bwd_rowterms_kernel<D>, dim3((unsigned)((threads + 255) / 256)), dim3(256), 0, stream, p,
                     rows);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  const BwdGrid grid = bwd_grid(D, p.BH, p.T);
  if (grid == BwdGrid::quads) return launch_grad<D, Quads<D>>(p, stream);
  if (grid == BwdGrid::pairs) return launch_grad<D, Pairs<D>>(p, stream);
  if constexpr (D == 64) {
    if (grid == BwdGrid::wide3) return launch_grad<D, Wide3>(p, stream);
  }
  return launch_grad<D, Wide<D>>(p, stream);
}

#if MW_BWD_HEAD_DIM == 128
int training_bwd_grid(int D, int BH, int T) { return (int)bwd_grid(D, BH, T); }
#endif

// This file is compiled once per head dimension (MW_BWD_HEAD_DIM = 64, 72 or 128):
// the two instantiations get different instruction-scheduling options in the
// build (each measured the faster one for its size).
#if MW_BWD_HEAD_DIM == 64
hipError_t launch_bwd_64(const BwdParams& p, hipStream_t stream) { return launch_bwd_d<64>(p, stream); }
#elif MW_BWD_HEAD_DIM == 72
hipError_t launch_bwd_72(const BwdParams& p, hipStream_t stream) { return launch_bwd_d<72>(p, stream); }
#elif MW_BWD_HEAD_DIM == 128
hipError_t launch_bwd_128(const BwdParams& p, hipStream_t stream) { return launch_bwd_d<128>(p, stream); }
#else
#error "compile with -DMW_BWD_HEAD_DIM=64, 72 or 128"
#endif

}  // namespace mw
