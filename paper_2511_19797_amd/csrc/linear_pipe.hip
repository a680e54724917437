// The linear layers' products (linear.hip says which) on 256 x 256 and 256 x 192 output tiles, hand-scheduled.
//
// Four waves, one per SIMD, as 2 x 2, each with 4 x 4 (4 x 3) blocks of 32 x 32: 256 (192) accumulators in AGPRs, and per
// contraction step of 16 eight (seven) fragments for 16 (12) products.  What binds a 256 x 256 tile of 64 contraction entries is
// LDS and L2 traffic next to 2048 cycles of matrix pipe: eight waves of 4 x 2 blocks read 192 KB of fragments from LDS for it, a
// CU's whole LDS rate with the 64 KB that land there, these four 128 KB.  A lone wave has nothing to hide behind but its own
// products, so the stream is laid out by hand (translation unit with the machine scheduler off: source order is issue order):
//   - fragments are read two steps ahead, one read every second product, the loads of later tiles in the slots between;
//   - one basic block per contraction tile: what a plain move to the next tile takes is a dozen scalar instructions dealt out
//     over the slots, anything else (ends of sets and of output tiles) happens every so many tiles (`quiet`);
//   - three P tiles (tokens, from HBM) and two Q tiles (weights, mostly in L2) in LDS: P is requested one and a half tiles ahead
//     of its barrier, Q one tile; with two of each the loop waited for what missed L2 (contraction tile of 256 x 192: 2400
//     cycles, now 1810; 1536 of them matrix pipe);
//   - operand rows of 128 bytes (64 contraction entries) in LDS, swizzled instead of padded: whole cache lines per request;
//   - loads are bounds-checked buffer loads: what lies outside arrives as zeros, with no code for ragged edges in the loop;
//   - results leave through LDS as whole cache lines (32-byte pieces straight from the accumulators: 4 x the requests to L2,
//     10 k cycles per output tile instead of 6 k), through chunks of the P slot that no one else touches at that time;
//   - tile positions by multiplication with reciprocals (five integer divisions per output tile were 3 k cycles).
// Accumulators start from bias x 1 as one more product, exactly the bias: every shape, these and the small ones, adds an output
// element's products in the same order.
// (The bias load is the newest of all when an output tile ends, and the compiler waits for it, in grad x without a bias too: the
// results' first store then stands behind every tile load in flight.  Grad W has no such wait.)
// Measured, DiT-XL/2 at 16 x 1024 tokens, against 8 waves of 4 x 2 blocks on tiles staged as 64-byte rows, us (TFLOP/s):
//   1152 -> 3456  forward 257 -> 225 (1160), grad x 287 -> 210 (1245), grad W 281 -> 211 (1235)
//   1152 -> 1152          94 ->  75 (1160),        105 ->  77 (1125),        102 ->  87 (1005)
//   1152 -> 4608         323 -> 281 (1240),        386 -> 271 (1285),        409 -> 286 (1215)
//   4608 -> 1152         390 -> 269 (1295),        322 -> 282 (1235),        421 -> 303 (1150)
// What bounds it now is power: with the loads and stores left out the same loop runs at 1.53 - 1.75 PFLOP/s, the matrix cores'
// limit on data; L2 -> LDS traffic costs 15 % on top, L2 misses 4 %, stores 7 %.
#include <type_traits>

#include "linear_gemm.h"
#include "pipe_ops.h"

namespace tvm {
namespace {

constexpr int kWI = 4;                         // 32-row blocks of a wave
constexpr unsigned kPTile = 32768;             // LDS: three P tiles, then two Q tiles

// Eight accumulator values, rounded to bf16.  (Assembly: plain conversions of all accumulators would be hoisted to one place;
// reads first, so that no conversion waits for the one before it.)
__device__ __forceinline__ void acc_to_bf16(unsigned& r0, unsigned& r1, unsigned& r2, unsigned& r3, float a0, float a1, float a2,
                                            float a3, float a4, float a5, float a6, float a7) {
  unsigned t0, t1, t2, t3;
  asm volatile(
      "v_accvgpr_read_b32 %0, %8\n\t"
      "v_accvgpr_read_b32 %4, %9\n\t"
      "v_accvgpr_read_b32 %1, %10\n\t"
      "v_accvgpr_read_b32 %5, %11\n\t"
      "v_accvgpr_read_b32 %2, %12\n\t"
      "v_accvgpr_read_b32 %6, %13\n\t"
      "v_accvgpr_read_b32 %3, %14\n\t"
      "v_accvgpr_read_b32 %7, %15\n\t"
      "v_cvt_pk_bf16_f32 %0, %0, %4\n\t"
      "v_cvt_pk_bf16_f32 %1, %1, %5\n\t"
      "v_cvt_pk_bf16_f32 %2, %2, %6\n\t"
      "v_cvt_pk_bf16_f32 %3, %3, %7"
      : "=&v"(r0), "=&v"(r1), "=&v"(r2), "=&v"(r3), "=&v"(t0), "=&v"(t1), "=&v"(t2), "=&v"(t3)
      : "a"(a0), "a"(a1), "a"(a2), "a"(a3), "a"(a4), "a"(a5), "a"(a6), "a"(a7));
}

// Slots of a contraction step: slot m is the gap behind its product m.  The NF fragment reads are spread over the slots from
// f0 on; the others are free for loads (once these run out, the n-th load takes one that is not).
template <int NP>
struct FreeSlots {
  int at[NP];
};
template <int NP, int NF>
constexpr FreeSlots<NP> free_slots(int f0) {
  FreeSlots<NP> s{};
  int n = 0;
  for (int m = f0; m < NP; ++m) {
    bool read = false;
    for (int f = 0; f < NF; ++f) read = read || m == f0 + f * (NP - f0) / NF;
    if (!read) s.at[n++] = m;
  }
  for (int m = f0 + 1; n < NP; m = m + 2 < NP ? m + 2 : f0) s.at[n++] = m;
  return s;
}

template <bool PTR, bool QTR, bool PARTIAL, int WJ>
__global__ __launch_bounds__(256, 1) void gemm_pipe_kernel(GemmArgs g) {
  constexpr int kTI = 256, kTJ = 64 * WJ;
  constexpr unsigned kQTile = kTJ * 128u;
  using OP = Operand<PTR, kTI>;
  using OQ = Operand<QTR, kTJ>;
  constexpr int NP = kWI * WJ;                 // products per contraction step
  constexpr int NF = kWI + WJ;                 // fragments per contraction step
  constexpr int LP = OP::LOADS, LQ = OQ::LOADS;
  constexpr int STORES = (PARTIAL ? 4 : 2) * NP;   // stores of a wave per output tile
  __shared__ __attribute__((aligned(1024))) char lds[3 * kPTile + 2 * kQTile];
  const int lane = threadIdx.x & 63, ic = lane & 31, hh = lane >> 5;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int wi = wave & 1, wj = wave >> 1;
  const unsigned lds0 = lds_addr_of(lds), ldsq = lds0 + 3 * kPTile;
  const int nI = (g.I + kTI - 1) / kTI, nJ = (g.J + kTJ - 1) / kTJ;
  const int nct = (g.C + 63) / 64, ntot = g.csets * nct;
  const int clast = g.C - (nct - 1) * 64;      // contraction entries in a set's last tile
  const unsigned pitchP = (unsigned)(g.ldP * 2), pitchQ = (unsigned)(g.ldQ * 2);

  // Persistent workgroups, one per CU, each working through a list of output tiles.  Hardware workgroup ids go round-robin over
  // the 8 XCDs, each with an L2 of its own: XCD x owns the x-th eighth of the logical tile ids, which its workgroups take in
  // turn; logical ids walk the tiles of a row set (or split) in groups of kGI tile rows, down the group first.  The 32
  // workgroups of an XCD are then on a patch of about 8 x 4 tiles at any one time and march through the contraction together:
  // an operand panel comes from HBM once for the tiles of the patch that share it.  (Groups of 4: the same; of 16: 4 % slower.)
  const int total = g.nz * nI * nJ;
  const int per_xcd = (total + 7) >> 3, wg_per_xcd = (int)(gridDim.x >> 3);
  const int id_end = min(total, ((int)(blockIdx.x & 7) + 1) * per_xcd);
  auto split_begin = [&](int z) {  // z * ntot / splits, as in gemm_small_kernel (splits <= 32, ntot <= 2^26)
    return (int)divide((unsigned)z * (unsigned)ntot, g.by_splits).q;
  };
  struct Where {
    int i0, j0, zz, t_begin, t_end;
  };
  auto locate = [&](int wg) {
    Where c;
    const Quotient z = divide((unsigned)wg, g.by_set), grp = divide(z.r, g.by_group);
    const int it_first = (int)grp.q * kGI;
    const Quotient jt = nI - it_first >= kGI ? Quotient{grp.r / kGI, grp.r % kGI} : divide(grp.r, g.by_rest);
    c.zz = (int)z.q;
    c.i0 = (it_first + (int)jt.r) * kTI;
    c.j0 = (int)jt.q * kTJ;
    c.t_begin = PARTIAL ? split_begin(c.zz) : 0;
    c.t_end = PARTIAL ? split_begin(c.zz + 1) : ntot;
    return c;
  };
  int wg = (int)(blockIdx.x & 7) * per_xcd + (int)(blockIdx.x >> 3);
  if (wg >= id_end) return;

  OP op;
  OQ oq;
  op.setup(lds0, wi, wave, lane, pitchP);
  oq.setup(ldsq, wj, wave, lane, pitchQ);

  // The loads run two contraction tiles ahead of the products, over the ends of output tiles.  The cursor is at the tile
  // they fetch; what changes from tile to tile within a segment (one contraction set of one output tile) is three additions
  // per operand, all else happens at its ends.
  u32x4 srd_p, srd_q;                       // descriptors: first byte, size for the bounds check
  unsigned vp[OP::NV], vq[OQ::NV];          // lane offsets
  int c_left, c_wg = wg, c_t, c_t_end;      // tiles left in the segment; output tile; tile behind the segment, last one
  bool c_ragged;                            // the segment ends with half a tile (row access)
  unsigned n_last_p, n_last_q;              // sizes of the segment's last tile (transposed access)
  auto open_one = [&](auto is_p, const Where& w, int set, int ct, bool to_end, u32x4& srd, unsigned& n_last) {
    constexpr bool P = decltype(is_p)::value, TR = P ? PTR : QTR;
    const long long c0 = (long long)ct * 64;
    const bf16* const m = P ? g.P[PARTIAL ? set : w.zz] : g.Q[set];
    const long long ld = P ? g.ldP : g.ldQ;
    const unsigned pitch = P ? pitchP : pitchQ;
    const int first = P ? w.i0 : w.j0, valid = P ? min(g.I - w.i0, kTI) : min(g.J - w.j0, kTJ);
    if (TR) {
      const unsigned n = 63u * pitch + (unsigned)valid * 2u;
      srd = descriptor((unsigned long long)(uintptr_t)(m + c0 * ld + first), n);
      n_last = to_end ? (unsigned)(clast - 1) * pitch + (unsigned)valid * 2u : n;
    } else {
      srd = descriptor((unsigned long long)(uintptr_t)(m + (long long)first * ld + c0),
                       (unsigned)(valid - 1) * pitch + (unsigned)(g.C - (int)c0) * 2u);
    }
  };
  const std::integral_constant<bool, true> is_p;
  const std::integral_constant<bool, false> is_q;
  auto lanes = [&]() {  // lane offsets of the cursor's tile
    const unsigned cut = c_left == 1 && c_ragged ? kNowhere : 0u;
    if (PTR && c_left == 1) srd_p[2] = n_last_p;
    if (QTR && c_left == 1) srd_q[2] = n_last_q;
#pragma unroll
    for (int k = 0; k < OP::NV; ++k) vp[k] = PTR ? op.voff[k] : op.voff[k] | (op.half & cut);
#pragma unroll
    for (int k = 0; k < OQ::NV; ++k) vq[k] = QTR ? oq.voff[k] : oq.voff[k] | (oq.half & cut);
  };
  auto open = [&](const Where& w, int t) {
    const int set = PARTIAL && t >= nct ? 1 : 0, ct = t - set * nct;
    const int end = min(w.t_end, (set + 1) * nct);
    const bool to_end = end == (set + 1) * nct;
    c_left = end - t;
    c_t = end;
    c_t_end = w.t_end;
    c_ragged = to_end && clast <= 32;
    open_one(is_p, w, set, ct, to_end, srd_p, n_last_p);
    open_one(is_q, w, set, ct, to_end, srd_q, n_last_q);
    lanes();
  };
  // the next tile of the segment
  auto further_p = [&]() {
    srd_p = descriptor(((unsigned long long)srd_p[1] << 32 | srd_p[0]) + (PTR ? 64ull * pitchP : 128ull), PTR ? srd_p[2] : srd_p[2] - 128u);
  };
  auto further_q = [&]() {
    srd_q = descriptor(((unsigned long long)srd_q[1] << 32 | srd_q[0]) + (QTR ? 64ull * pitchQ : 128ull), QTR ? srd_q[2] : srd_q[2] - 128u);
  };
  auto advance = [&]() {  // behind further_p, further_q: where the segment goes on differently, or has ended
    if (--c_left > 0) {
      lanes();
    } else if (PARTIAL && c_t < c_t_end) {
      open(locate(c_wg), c_t);
    } else if (c_wg + wg_per_xcd < id_end) {
      c_wg += wg_per_xcd;
      const Where w = locate(c_wg);
      open(w, w.t_begin);
    } else {  // nothing more: size 0, loads that fetch nothing, so that the count of loads in flight stays the same
      srd_p = srd_q = descriptor(0, 0);
      c_left = 1;
      c_wg = id_end;
    }
  };
  unsigned slot_p = lds0 + (unsigned)wave * 1024u, slot_q = ldsq + (unsigned)wave * 1024u;  // where the next tile's loads go
  auto issue_p = [&](int x) {
    load_lds(srd_p, vp[x % OP::NV], (unsigned)(x / OP::NV * OP::ROWS_STEP) * pitchP, slot_p, x * 4096);
  };
  auto issue_q = [&](int x) {
    load_lds(srd_q, vq[x % OQ::NV], (unsigned)(x / OQ::NV * OQ::ROWS_STEP) * pitchQ, slot_q, x * 4096);
  };

  f32x16 acc[kWI][WJ];
  bf16x8 pf[4][kWI], qf[4][WJ];
  auto fetch = [&](int kk, int f) {  // fragment number f of contraction step kk of the tile at the read addresses
    if (f < WJ) qf[kk][f] = oq.frag(f, kk);
    else pf[kk][f - WJ] = op.frag(f - WJ, kk);
  };

  // bias of the wave's columns (row set 0 only): block b's column 32 b + ic
  unsigned bias_bits[WJ];
  auto bias_load = [&](const Where& w) {
    const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<bf16*>(g.bias), 0, g.bias != nullptr && w.zz == 0 ? g.J * 2 : 0, 0x00027000);
#pragma unroll
    for (int b = 0; b < WJ; ++b) {
      const unsigned off = (unsigned)(w.j0 + (wj * WJ + b) * 32 + ic) * 2u;
      bias_bits[b] = PARTIAL ? 0u : (unsigned)(unsigned short)__builtin_amdgcn_raw_buffer_load_b16(rs, (int)(hh == 0 ? off : kNowhere), 0, 0);
    }
  };
  const unsigned one_bits = hh == 0 ? 0x3f80u : 0u;  // bf16 1.0
  auto start = [&](int a) {  // accumulators of block row a start from bias (x) 1, exactly the bias
    const bf16x8 one = __builtin_bit_cast(bf16x8, u32x4{one_bits, 0u, 0u, 0u});
#pragma unroll
    for (int b = 0; b < WJ; ++b) {
      const bf16x8 bv = __builtin_bit_cast(bf16x8, u32x4{bias_bits[b], 0u, 0u, 0u});
      asm volatile("s_nop 1\n\tv_mfma_f32_32x32x16_bf16 %0, %1, %2, 0" : "+a"(acc[a][b]) : "v"(bv), "v"(one));
    }
  };

  auto start_after = [&](int n, int a, int ns) {  // once a block row's last piece is out of the accumulators
    if (n % ns == ns - 1) start(a);
  };
  // Results of output tile w: [32 rows x 128 bytes] at a time (two blocks of bf16, one of float32; a last single block of bf16:
  // 64 bytes a row) through LDS, so that they leave as whole cache lines.  The place: the P tile that was just worked on is
  // free, and of the slot that the next P tile goes to, the chunks that this wave's own loads will fill are its own: 1 KB every
  // 4 KB.  A chunk holds 8 rows (16 of 64 bytes); 16-byte chunks within them are swizzled, and in rows 16 to 31 the 8-byte
  // halves that the two half-waves write change places, so that no two lanes meet in a bank.
  typedef __attribute__((ext_vector_type(2))) unsigned u32x2;
  typedef __attribute__((ext_vector_type(4))) float f32x4;
  auto write_out = [&](const Where& w) {
    typedef u32x2 __attribute__((address_space(3))) * wp2;
    typedef f32x4 __attribute__((address_space(3))) * wp4;
    typedef const u32x4 __attribute__((address_space(3))) * rp;
    const int i_first = w.i0 + wi * (kWI * 32), j_first = w.j0 + wj * (WJ * 32);
    const int rows = max(0, min(g.I - i_first, kWI * 32)), cols = max(0, min(g.J - j_first, WJ * 32));
    constexpr int E = PARTIAL ? 4 : 2;
    const unsigned pitch = PARTIAL ? (unsigned)g.J * 4u : (unsigned)(g.ldo * 2);
    char* const base = PARTIAL ? reinterpret_cast<char*>(g.part + (long long)w.zz * g.I * g.J + (long long)i_first * g.J + j_first)
                               : reinterpret_cast<char*>(g.out[w.zz] + (long long)i_first * g.ldo + j_first);
    const int bytes = rows > 0 && cols > 0 ? (int)((unsigned)(rows - 1) * pitch + (unsigned)cols * E) : 0;
    const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(base, 0, bytes, 0x00027000);
    constexpr int WB = PARTIAL ? 1 : 2;               // blocks of a piece
    constexpr int NS = (WJ + WB - 1) / WB;            // pieces per block row
    const unsigned at128 = slot_p + (unsigned)(ic >> 3) * 4096u + (unsigned)(ic & 7) * 128u, sw128 = (unsigned)(ic >> 1) & 7u;
    const unsigned at64 = slot_p + (unsigned)(ic >> 4) * 4096u + (unsigned)(ic & 15) * 64u, sw64 = (unsigned)(ic >> 2) & 3u;
    const unsigned half = (unsigned)(hh ^ (ic >> 4)) * 8u;
    // read side: lane -> row r8 of 8 (16), chunk
    const unsigned rd128 = slot_p + (unsigned)(lane >> 3) * 128u, rd64 = slot_p + (unsigned)(lane >> 2) * 64u;
    const unsigned out128 = (unsigned)(lane >> 3) * pitch + (unsigned)(lane & 7) * 16u, out64 = (unsigned)(lane >> 2) * pitch + (unsigned)(lane & 3) * 16u;
    u32x4 v[4];
    auto park = [&](int n) __attribute__((always_inline)) {     // piece n into its half of the place
      const int a = n / NS, b0 = n % NS * WB, nb = WJ - b0 < WB ? WJ - b0 : WB;
      const unsigned buf = (unsigned)(n & 1) * 16384u;
      for (int b = b0; b < b0 + nb; ++b) {
        const f32x16& t = acc[a][b];
        if constexpr (PARTIAL) {
#pragma unroll
          for (int q4 = 0; q4 < 4; ++q4)
            *(wp4)(uintptr_t)(at128 + buf + (((unsigned)(2 * q4 + hh)) ^ sw128) * 16u) = f32x4{t[4 * q4], t[4 * q4 + 1], t[4 * q4 + 2], t[4 * q4 + 3]};
        } else {
#pragma unroll
          for (int h = 0; h < 2; ++h) {
            unsigned r0, r1, r2, r3;
            acc_to_bf16(r0, r1, r2, r3, t[8 * h], t[8 * h + 1], t[8 * h + 2], t[8 * h + 3], t[8 * h + 4], t[8 * h + 5],
                        t[8 * h + 6], t[8 * h + 7]);
            const unsigned c = (unsigned)((b - b0) * 4 + 2 * h);
            const unsigned at = (nb == 2 ? at128 : at64) + buf + half, sw = nb == 2 ? sw128 : sw64;
            *(wp2)(uintptr_t)(at + (c ^ sw) * 16u) = u32x2{r0, r1};
            *(wp2)(uintptr_t)(at + ((c + 1) ^ sw) * 16u) = u32x2{r2, r3};
          }
        }
      }
      start_after(n, a, NS);
    };
    auto fetch_back = [&](int n) __attribute__((always_inline)) {
      const bool wide = PARTIAL || n % NS * WB + WB <= WJ;
      const unsigned buf = (unsigned)(n & 1) * 16384u;
#pragma unroll
      for (int it = 0; it < (wide ? 4 : 2); ++it) {
        const unsigned sw = wide ? (unsigned)(4 * it + (lane >> 4)) & 7u : (unsigned)(lane >> 4) & 3u;  // (row >> 1) & 7, (row >> 2) & 3
        v[it] = *(rp)(uintptr_t)((wide ? rd128 : rd64) + buf + (unsigned)it * 4096u + (((unsigned)(wide ? lane & 7 : lane & 3)) ^ sw) * 16u);
      }
    };
    auto store = [&](int n) __attribute__((always_inline)) {
      const int a = n / NS, b0 = n % NS * WB;
      const bool wide = PARTIAL || b0 + WB <= WJ;
      // (widths are multiples of 32; a lane's 16 bytes are in range together)
      const bool in = b0 * 32 * E + (wide ? lane & 7 : lane & 3) * 16 < cols * E;
#pragma unroll
      for (int it = 0; it < (wide ? 4 : 2); ++it) {
        const bool swapped = !PARTIAL && it >= (wide ? 2 : 1);
        const u32x4 o = swapped ? u32x4{v[it][2], v[it][3], v[it][0], v[it][1]} : v[it];
        const unsigned off = (wide ? out128 : out64) + (unsigned)(a * 32 + it * (wide ? 8 : 16)) * pitch + (unsigned)(b0 * 32 * E);
        __builtin_amdgcn_raw_buffer_store_b128(o, rs, (int)(in ? off : kNowhere), 0, 0);
      }
    };
    park(0);
    fetch_back(0);
#pragma unroll
    for (int n = 1; n < kWI * NS; ++n) {
      park(n);
      store(n - 1);
      fetch_back(n);
    }
    store(kWI * NS - 1);
  };

  // Start: tiles 0 and 1 on their way, the accumulators from the bias, the first fragments.
  Where w = locate(wg);
  bias_load(w);
  open(w, w.t_begin);
#pragma unroll
  for (int n = 0; n < 2; ++n) {
#pragma unroll
    for (int x = 0; x < LP; ++x) issue_p(x);
#pragma unroll
    for (int x = 0; x < LQ; ++x) issue_q(x);
    slot_p += kPTile;
    slot_q += n == 0 ? kQTile : 0u - kQTile;
    further_p();
    further_q();
    advance();
  }
  asm volatile("s_waitcnt vmcnt(%0)\n\ts_barrier" ::"n"(LP + LQ) : "memory");
#pragma unroll
  for (int a = 0; a < kWI; ++a) start(a);
#pragma unroll
  for (int f = 0; f < NF; ++f) fetch(0, f);
#pragma unroll
  for (int f = 0; f < NF; ++f) fetch(1, f);
  int left = w.t_end - w.t_begin;      // contraction tiles of this output tile yet to be worked on
  int quiet = 1, passed = 1;           // tiles until something other than further() is due, and their number
  // byte offsets of the P tile being read and the next one; from the Q tile being read to the other one
  unsigned p_now = 0, p_next = kPTile, q_step = kQTile;
  int fresh = 0;                       // results left in front of this tile
  for (;;) {
    // Products of contraction step kk.  Behind product m: the fragments of step kk + 2, and the loads of the tile two ahead
    // (P in steps 0 and 1, Q in steps 2 and 3), in slots without fragment reads.
    auto step = [&](auto kkc) {
      constexpr int kk = decltype(kkc)::value;
      constexpr int sync = 1;                          // step 2: the barrier's slot
      constexpr int f0 = kk == 2 ? sync + 1 : 0;       // first slot with fragment reads (step 2: behind the barrier)
      constexpr FreeSlots<NP> slots = free_slots<NP, NF>(f0);
      constexpr int nfree = NP - f0 - NF, L = kk < 2 ? LP / 2 : LQ / 2, x0 = (kk & 1) * L;
#pragma unroll
      for (int m = 0; m < NP; ++m) {
        mfma_acc(acc[m / WJ][m % WJ], qf[kk][m % WJ], pf[kk][m / WJ]);
        if (kk == 2 && m == sync) {
          // Everyone has read its last fragments of this tile, and the next tile is there for everyone.  Younger than its
          // loads: the stores of an output tile's results, and the loads of the P tile behind it.  (Branch in the assembly:
          // the tile stays one basic block, over which the compiler keeps the order.)
          asm volatile(
              "s_cmp_lg_u32 %0, 0\n\t"
              "s_cbranch_scc1 .Ltvm_fresh_%=\n\t"
              "s_waitcnt vmcnt(%1)\n"
              ".Ltvm_fresh_%=:\n\t"
              "s_waitcnt vmcnt(%2) lgkmcnt(0)\n\t"
              "s_barrier" ::"s"(__builtin_amdgcn_readfirstlane(fresh)), "n"(LP), "n"(LP + STORES < 63 ? LP + STORES : 63)
              : "memory", "scc");
          op.move(p_next - p_now);
          oq.move(q_step);
        }
#pragma unroll
        for (int f = 0; f < NF; ++f)
          if (m == f0 + f * (NP - f0) / NF) fetch((kk + 2) & 3, f);
#pragma unroll
        for (int x = 0; x < L; ++x)
          if (m == slots.at[x * nfree / L]) {
            if (kk < 2) issue_p(x0 + x);
            else issue_q(x0 + x);
          }
        if (kk == 3 && m == 2) {  // the bookkeeping of a plain move to the next tile, in slots that have room
          const unsigned p_free = 3 * kPTile - p_now - p_next;
          slot_p += p_now - p_free;
          p_now = p_next;
          p_next = p_free;
          fresh = 0;
        }
        if (kk == 3 && m == NP / 2) further_p();
        if (kk == 3 && m == NP - 2) {
          slot_q += q_step;
          q_step = 0u - q_step;
          further_q();
        }
      }
    };
    step(std::integral_constant<int, 0>{});
    step(std::integral_constant<int, 1>{});
    step(std::integral_constant<int, 2>{});
    step(std::integral_constant<int, 3>{});
    if (--quiet == 0) {
      c_left -= passed - 1;
      left -= passed;
      advance();
      // the cursor's moves are plain until it reaches the segment's last tile
      passed = quiet = max(1, c_left - 2);
      if (left > 0) passed = quiet = min(quiet, left);
      __builtin_amdgcn_s_waitcnt(0xc07f);  // scalar loads, here: with one on its way the fragments behind would all be waited for
    }
    if (left == 0) {
      const Where nw = locate(min(wg + wg_per_xcd, id_end - 1));
      bias_load(nw);
      mfma_settle();
      write_out(locate(wg));
      fresh = 1;
      wg += wg_per_xcd;
      if (wg >= id_end) break;
      left = nw.t_end - nw.t_begin;
      passed = quiet = min(quiet, left);
      __builtin_amdgcn_s_waitcnt(0xc07f);
    }
  }
  dma_wait();  // (no load may land in LDS that the next workgroup owns)
}

// Persistent workgroups: 8 XCDs x at most 32 CUs, fewer where an XCD's share of the tiles is smaller.
int persistent_grid(int tiles) {
  const int per = (tiles + 7) / 8;
  return 8 * (per < 32 ? per : 32);
}
template <bool PTR, bool QTR, bool PARTIAL>
hipError_t launch(int shape, GemmArgs g, hipStream_t st) {
  g.set_divisors(shape, PARTIAL);
  const dim3 grid(persistent_grid((int)(g.nz * tiles_of(shape, g.I, g.J))));
  if (shape == k192) hipLaunchKernelGGL((gemm_pipe_kernel<PTR, QTR, PARTIAL, 3>), grid, dim3(256), 0, st, g);
  else hipLaunchKernelGGL((gemm_pipe_kernel<PTR, QTR, PARTIAL, 4>), grid, dim3(256), 0, st, g);
  return hipGetLastError();
}
static_assert(kTileI[k256] == 256 && kTileJ[k256] == 256 && kTileI[k192] == 256 && kTileJ[k192] == 192 && kBK == 64, "the plan's tiles");

}  // namespace

hipError_t launch_gemm_fwd(int shape, const GemmArgs& g, hipStream_t st) { return launch<false, false, false>(shape, g, st); }
hipError_t launch_gemm_gx(int shape, const GemmArgs& g, hipStream_t st) { return launch<false, true, false>(shape, g, st); }
hipError_t launch_gemm_gw(int shape, const GemmArgs& g, hipStream_t st) { return launch<true, true, true>(shape, g, st); }

}  // namespace tvm
