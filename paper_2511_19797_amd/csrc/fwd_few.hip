// Forward with tangent on the bf16 matrix cores for few query rows (the mathematics, fragments and tiles of
// fwd_mfma.hip).
//
// There a workgroup owns 128 or 256 query rows and walks all keys: one head of 4096 rows is 16 workgroups on 256 CUs,
// bound by the length of that walk.  Here a workgroup owns 32 query rows and its four waves deal the tiles of 32 keys out
// among themselves, each with a running maximum and accumulators of its own, which meet through LDS at the end:
// eight times the workgroups and a quarter of the walk, for operand tiles fetched once per 32 rows (from L2) instead of once
// per 256.  A wave fetches its own tiles (no barrier in the loop) into one stage: the fragments of K, tK are read to
// registers first and the next tile's K, tK requested behind them, those of V, tV likewise, so that each half of the stage
// has the other half's work to land behind.
// Bound by the products and the softmax of one wave per SIMD.  One head of 4096, d = 64 (128 workgroups): 136 us on 16 workgroups
// of fwd_mfma.hip, 32 us here (200 TFLOP/s on half of the CUs).
#include "fwd_few.h"
#include "mfma_tiles.h"

namespace tvm {
namespace {

constexpr float kLog2e = 1.4426950408889634f;
constexpr float kRescaleLog2 = 8.f;  // raise the reference maximum only beyond this growth (log2 units), as in fwd_mfma.hip
constexpr int kNW = 4;               // waves per workgroup

// LDS reads issued so far have returned: what they read from may be refilled.
__device__ __forceinline__ void lds_reads_done() { asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory"); }

template <int DK, int DV, bool SPARE>
__global__ __launch_bounds__(64 * kNW, 1) void fwd_few_kernel(Shape s, const bf16* __restrict__ q, const bf16* __restrict__ k,
                                                              const bf16* __restrict__ v, const bf16* __restrict__ tq,
                                                              const bf16* __restrict__ tk, const bf16* __restrict__ tv,
                                                              bf16* __restrict__ o, bf16* __restrict__ to,
                                                              float* __restrict__ lse, float* __restrict__ stats) {
  typedef __attribute__((ext_vector_type(4))) float f32x4;
  using TK = Tile<32, DK / 8, 1>;
  using TV = Tile<32, DV / 8, 1>;
  constexpr int NKS = DK / 16, NDB = DV / 32;
  constexpr int BUF = 2 * TK::BYTES + 2 * TV::BYTES;  // a wave's stage: K, tK, V, tV
  constexpr int ACC = 2 * NDB * 16 * 64 * 4;          // a wave's accumulators, float32
  constexpr int OFF_OUT = kNW * ACC, OUT_REGION = 32 * (64 + 16), OFF_ROW = OFF_OUT + kNW * OUT_REGION;
  constexpr int END = OFF_ROW + kNW * 3 * 32 * 4;     // behind the loop: accumulators, output staging, row scalars
  constexpr int LDS_BYTES = kNW * BUF > END ? kNW * BUF : END;
  static_assert(LDS_BYTES <= 160 * 1024, "LDS of a CU");
  __shared__ __attribute__((aligned(16))) char lds[LDS_BYTES];
  const int tid = threadIdx.x, lane = tid & 63, ic = lane & 31, hh = lane >> 5;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int nmb = (s.M + 31) / 32;
  const int wg = xcd_remap(blockIdx.x, gridDim.x);
  const int bh = wg / nmb, mb = wg - bh * nmb;
  const int b = bh / s.H, h = bh - b * s.H;
  const long long base = b * s.sb + h * s.sh;     // key side
  const long long qbase = b * s.qsb + h * s.qsh;  // query side
  const int i = mb * 32 + ic;                     // this lane's query row
  const unsigned pitch = (unsigned)(s.sn * 2);
  char* const mine = lds + wave * BUF;
  const unsigned lds0 = lds_addr_of(lds), st = lds0 + (unsigned)wave * BUF;
  const int ntiles = (int)(((unsigned)s.N + 31u) >> 5), tlast = ntiles - 1;
  // per-lane byte offsets of the loads within a tile: for whole tiles, and for the last one, where rows past the end
  // fetch its last row again (keys of probability 0)
  typename TK::Offs ok_full, ok_last;
  typename TV::Offs ov_full, ov_last;
  {
    const typename TK::Lane lk = TK::lane_setup(s.D, 0, lane);
    const typename TV::Lane lv = TV::lane_setup(s.D, 0, lane);
    ok_full = TK::offsets(lk, pitch, 32);
    ok_last = TK::offsets(lk, pitch, s.N - tlast * 32);
    ov_full = TV::offsets(lv, pitch, 32);
    ov_last = TV::offsets(lv, pitch, s.N - tlast * 32);
  }
  constexpr int LK = 2 * TK::IPW, LV = 2 * TV::IPW;  // loads of K, tK and of V, tV per tile
  auto issue_k = [&](int t) {
    const long long ro = base + (long long)t * 32 * s.sn;
#pragma unroll
    for (int x = 0; x < TK::IPW; ++x) {
      const unsigned off = t == tlast ? ok_last.o[x] : ok_full.o[x];
      TK::issue_at(off, x, k + ro, st, 0);
      TK::issue_at(off, x, tk + ro, st + TK::BYTES, 0);
    }
  };
  auto issue_v = [&](int t) {
    const long long ro = base + (long long)t * 32 * s.sn;
#pragma unroll
    for (int x = 0; x < TV::IPW; ++x) {
      const unsigned off = t == tlast ? ov_last.o[x] : ov_full.o[x];
      TV::issue_at(off, x, v + ro, st + 2 * TK::BYTES, 0);
      TV::issue_at(off, x, tv + ro, st + 2 * TK::BYTES + TV::BYTES, 0);
    }
  };
  const typename TK::RAddr rk = TK::raddr(ic, hh);
  const typename TV::TAddr ta = TV::taddr(ic, hh);
  // the query rows first: the compiler's waits for them count every load in flight
  bf16x8 qf[NKS], tqf[NKS];
  {
    uint4 w0[NKS], w1[NKS];
    gld_frags_issue<NKS>(w0, q + qbase, s.qsn, i, s.M, s.D, hh);
    gld_frags_issue<NKS>(w1, tq + qbase, s.qsn, i, s.M, s.D, hh);
    gld_frags_finish<NKS>(qf, w0, i, s.M, s.D, hh);
    gld_frags_finish<NKS>(tqf, w1, i, s.M, s.D, hh);
  }
  pin_frags(qf);
  pin_frags(tqf);
  f32x16 accO[NDB], accT[NDB];
#pragma unroll
  for (int db = 0; db < NDB; ++db) {
    accO[db] = zero16();
    accT[db] = zero16();
  }
  float m = -INFINITY, l = 0.f, cs = 0.f;
  const float c1 = s.alpha * kLog2e;  // scores are exponentiated in base 2
  // SPARE: column D of the wave's V rows is set to one and of its tV rows to zero once they have landed (fwd_mfma.hip)
  char* const plant = mine + (hh ? 2 * TK::BYTES + TV::BYTES : 2 * TK::BYTES) + (ic * TV::PCH + ((s.D >> 3) ^ ((ic >> 2) & 3))) * 16;

  if (wave < ntiles) {  // uniform in a wave; the loop has no barrier
    issue_k(wave);
    issue_v(wave);
    for (int t = wave; t < ntiles; t += kNW) {
      const int tn = min(t + kNW, tlast);  // (behind the wave's last tile: a tile that is fetched and not used)
      dma_wait_keep<LV>();                 // K, tK of this tile
      bf16x8 kf[NKS], tkf[NKS];
#pragma unroll
      for (int kk = 0; kk < NKS; ++kk) {
        kf[kk] = TK::frag_row(mine, rk, 0, kk);
        tkf[kk] = TK::frag_row(mine + TK::BYTES, rk, 0, kk);
      }
      pin_frags(kf);
      pin_frags(tkf);
      lds_reads_done();
      issue_k(tn);
      f32x16 sS = zero16(), sT = zero16();
#pragma unroll
      for (int kk = 0; kk < NKS; ++kk) {
        sS = mfma(kf[kk], qf[kk], sS);
        sT = mfma(kf[kk], tqf[kk], sT);
        sT = mfma(tkf[kk], qf[kk], sT);
      }
      if (s.N - t * 32 < 32) {  // uniform: ragged last tile, keys >= N get probability 0
#pragma unroll
        for (int r = 0; r < 16; ++r)
          if (drow(r, hh) >= s.N - t * 32) sS[r] = -INFINITY;
      }
      float mx = sS[0];
#pragma unroll
      for (int r = 1; r < 16; ++r) mx = fmaxf(mx, sS[r]);
      mx = fmaxf(mx, xhalf(mx));
      if (__builtin_amdgcn_ballot_w64((mx - m) * c1 > kRescaleLog2) != 0) {  // uniform
        const float mn = fmaxf(m, mx);
        const float f = m == -INFINITY ? 0.f : __builtin_amdgcn_exp2f((m - mn) * c1);
        m = mn;
        if (!SPARE) {
          l *= f;
          cs *= f;
        }
#pragma unroll
        for (int db = 0; db < NDB; ++db)
#pragma unroll
          for (int r = 0; r < 16; ++r) {
            accO[db][r] *= f;
            accT[db][r] *= f;
          }
      }
      // (a wave may see no key of finite score so far, another one will: its weights are then zero, not exp(-inf + inf))
      const float mc = m == -INFINITY ? 0.f : m * c1;
      bf16x8 pf[2], pzf[2];
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const float p = __builtin_amdgcn_exp2f(fmaf(sS[r], c1, -mc));
        const float pz = p * (sT[r] * s.alpha);
        if (!SPARE) {
          l += p;  // per-half sums; the halves are combined behind the loop
          cs += pz;
        }
        pf[r >> 3][r & 7] = (bf16)p;
        pzf[r >> 3][r & 7] = (bf16)pz;
      }
      dma_wait_keep<LK>();  // V, tV of this tile
      if (SPARE) *reinterpret_cast<uint4*>(plant) = make_uint4(hh ? 0u : 0x3F80u, 0u, 0u, 0u);
      const char* const lv = mine + 2 * TK::BYTES;
      bf16x8 vf[2][NDB], tvf[2][NDB];
#pragma unroll
      for (int c = 0; c < 2; ++c) {
#pragma unroll
        for (int db = 0; db < NDB; ++db) {
          vf[c][db] = TV::frag_tr(lv, ta, c, db);
          tvf[c][db] = TV::frag_tr(lv + TV::BYTES, ta, c, db);
        }
        pin_frags(vf[c]);
        pin_frags(tvf[c]);
      }
      lds_reads_done();
      issue_v(tn);
#pragma unroll
      for (int c = 0; c < 2; ++c)
#pragma unroll
        for (int db = 0; db < NDB; ++db) {
          accO[db] = mfma(vf[c][db], pf[c], accO[db]);
          accT[db] = mfma(vf[c][db], pzf[c], accT[db]);
          accT[db] = mfma(tvf[c][db], pf[c], accT[db]);
        }
    }
  }
  if (SPARE) {  // row D of the accumulators (held by the lower half-wave) has the sums
    float lv = 0.f, cv = 0.f;
#pragma unroll
    for (int cand = DK - 8; cand <= DK; cand += 8)
      if (cand < DV && s.D == cand) {
        lv = accO[cand / 32][4 * ((cand % 32) / 8)];
        cv = accT[cand / 32][4 * ((cand % 32) / 8)];
      }
    const float lx = xhalf(lv), cx = xhalf(cv);
    l = hh ? lx : lv;
    cs = hh ? cx : cv;
  } else {
    l += xhalf(l);
    cs += xhalf(cs);
  }
  // The four waves meet: the common maximum first, then everything scaled to it.
  dma_wait();  // the tiles fetched and not used are over before their place is written to
  __syncthreads();
  float* const rows = reinterpret_cast<float*>(lds + OFF_ROW);  // [m, l, cs][wave][32]
  if (hh == 0) rows[wave * 32 + ic] = m;
  __syncthreads();
  float mt = rows[ic];
#pragma unroll
  for (int w = 1; w < kNW; ++w) mt = fmaxf(mt, rows[w * 32 + ic]);
  const float f = m == -INFINITY && mt != -INFINITY ? 0.f : __builtin_amdgcn_exp2f((m - mt) * c1);
  if (hh == 0) {
    rows[(kNW + wave) * 32 + ic] = l * f;
    rows[(2 * kNW + wave) * 32 + ic] = cs * f;
  }
  // [wave][O, T][db][group of four rows][lane] four floats
  f32x4* const accs = reinterpret_cast<f32x4*>(lds);
  constexpr int WACC = ACC / 16;
#pragma unroll
  for (int db = 0; db < NDB; ++db)
#pragma unroll
    for (int g = 0; g < 4; ++g) {
      const f32x4 vo = {accO[db][4 * g], accO[db][4 * g + 1], accO[db][4 * g + 2], accO[db][4 * g + 3]};
      const f32x4 vt = {accT[db][4 * g], accT[db][4 * g + 1], accT[db][4 * g + 2], accT[db][4 * g + 3]};
      accs[wave * WACC + (db * 4 + g) * 64 + lane] = vo * f;
      accs[wave * WACC + ((NDB + db) * 4 + g) * 64 + lane] = vt * f;
    }
  __syncthreads();
  l = cs = 0.f;
#pragma unroll
  for (int w = 0; w < kNW; ++w) {
    l += rows[(kNW + w) * 32 + ic];
    cs += rows[(2 * kNW + w) * 32 + ic];
  }
  const float inv = 1.f / l;
  const float mubar = cs * inv;
  const float nmi = -mubar * inv;
  static_assert(NDB <= kNW, "a wave for every block of 32 columns");
  if (wave < NDB) {
    f32x16 aO[1], aT[1];
#pragma unroll
    for (int g = 0; g < 4; ++g) {
      f32x4 vo = {0.f, 0.f, 0.f, 0.f}, vt = vo;
#pragma unroll
      for (int w = 0; w < kNW; ++w) {
        vo += accs[w * WACC + (wave * 4 + g) * 64 + lane];
        vt += accs[w * WACC + ((NDB + wave) * 4 + g) * 64 + lane];
      }
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        aO[0][4 * g + e] = vo[e];
        aT[0][4 * g + e] = fmaf(nmi, vo[e], vt[e] * inv);
      }
    }
    const unsigned lw = lds0 + OFF_OUT + (unsigned)wave * OUT_REGION;
    store_tile_coalesced<1>(lw, o + qbase + wave * 32, s.qsn, mb * 32, s.M, s.D - wave * 32, aO, inv, lane);
    store_tile_coalesced<1>(lw, to + qbase + wave * 32, s.qsn, mb * 32, s.M, s.D - wave * 32, aT, 1.f, lane);
  }
  if (wave == 0 && i < s.M && hh == 0) {
    const long long r = (long long)bh * s.M + i;
    if (lse) lse[r] = (mt * c1 + __builtin_amdgcn_logf(l)) * 0.6931471805599453f;
    if (stats) stats[r] = mubar;
  }
}

template <int DK, int DV>
hipError_t launch(const Shape& s, const FwdArgs& a, hipStream_t st) {
  const dim3 grid((s.M + 31) / 32 * s.B * s.H), block(64 * kNW);
  auto go = [&](auto kernel) {
    hipLaunchKernelGGL(kernel, grid, block, 0, st, s, (const bf16*)a.q, (const bf16*)a.k, (const bf16*)a.v, (const bf16*)a.tq,
                       (const bf16*)a.tk, (const bf16*)a.tv, (bf16*)a.o, (bf16*)a.to, a.lse, a.stats);
    return hipGetLastError();
  };
  if (s.D < DV) return go(fwd_few_kernel<DK, DV, true>);
  if constexpr (DK == DV) return go(fwd_few_kernel<DK, DV, false>);
  return hipErrorNotSupported;  // D <= DK < DV: not reached
}

}  // namespace

hipError_t launch_fwd_few(const Shape& s, const FwdArgs& a, hipStream_t st) {
  switch ((s.D + 15) / 16 * 16) {
    case 16: return launch<16, 32>(s, a, st);
    case 32: return launch<32, 32>(s, a, st);
    case 48: return launch<48, 64>(s, a, st);
    case 64: return launch<64, 64>(s, a, st);
    case 80: return launch<80, 96>(s, a, st);
    case 96: return launch<96, 96>(s, a, st);
    case 112: return launch<112, 128>(s, a, st);
    case 128: return launch<128, 128>(s, a, st);
    default: return hipErrorNotSupported;
  }
}

}  // namespace tvm
