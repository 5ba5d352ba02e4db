// Gated prefill / training forward of libeta for gfx950 (CDNA4, wave64):
// causal attention over gated scores, with the per-row gate sums R and the
// log-sum-exp L (paper: "Elastic Threshold Attention", App. "Hardware-Aligned
// Forward Kernel", Alg. fwd_kernel).  fp32 accumulation, bf16 operands.

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

#include "eta_device.h"
#include "eta_internal.h"

namespace eta {
namespace {

// ---------------------------------------------------------------- gated prefill forward
//
// The training / prefill forward (App. "Hardware-Aligned Forward Kernel"):
// causal attention over gated scores S~ = S sigma(beta (S - tau_i)) (or the
// additive S + C sigma - C), diagonal ungated, with the gate row sums R and the
// log-sum-exp L.  One workgroup per (128-query block, query head, sequence);
// wavefront w owns query rows 32 w .. 32 w + 31.  Everything is computed
// transposed so that each lane owns one query row: S^T = K Q^T on
// v_mfma_f32_32x32x16_bf16 (A = 32 keys x 16 dims from LDS, B = 16 dims x 32
// queries from registers) gives lane l the scores of query l & 31 against keys
// 8 (i / 4) + 4 (l / 32) + i % 4 of each 32-key half; the gate, mask and online
// softmax are per lane (lanes l and l ^ 32 share a row); O^T += V^T P^T takes
// B = the lane's own gated weights (bf16), the contraction over keys permuted
// consistently on both sides, and A = V^T from two LDS transpose reads
// (ds_read_b64_tr_b16) of the row-major V tile.  fp32 accumulators.
//
// What bounds it: vector-ALU issue (a score takes three transcendentals, two
// issue slots each, and six other instructions; the MFMAs need half of that
// time), and at 16K tokens the card's power: the clock drops to about 1.9 GHz
// under the overlapped load.  So the matrix work is threaded through the vector work of the
// same wavefront, in units of 32 keys: beside unit u's gates and weights run unit
// u - 1's p.V MFMAs and unit u + 1's score MFMAs, in an order fixed by scheduling
// barriers.  32x32x16 MFMAs: the rate of 16x16x32 ones at half the instructions,
// each of which takes issue slots from the vector work (measured on single
// instruction streams: about 5 cycles per MFMA of either shape), and one
// query row per lane halves the row bookkeeping.  Measured against the kernel
// before it (16x16x32, scores, softmax and p.V one after the other): 16K tokens,
// 32/8 heads, d = 128: 3.34 -> 2.48 ms (659 -> 887 TFLOP/s); 2048 tokens, 128
// heads, d = 64: 269 -> 131 us, d = 128: 333 -> 194 us, where the workgroup order
// below also evens out the XCDs.  Tried: 64-key units (all 256 registers, no faster; 3.7
// ms with p.V carried into the next unit, which spills); eight wavefronts sharing the
// tiles, 256 rows (half the L2 reads, but both wavefronts of a SIMD then wait at one
// barrier: 1% faster at 16K, 18% slower at 2000 tokens).

constexpr int kPfQ = 128;    // query rows per workgroup (32 per wavefront)
constexpr int kPfK = 64;     // keys per block

struct PrefillArgs {
  const uint16_t* q;
  const uint16_t* k;
  const uint16_t* v;
  const float* tau;
  const int32_t* seq_lens;
  uint16_t* out;
  float* R;
  float* L;
  int Hq, Hkv, T;
  float beta, C;
};

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef short i16x4 __attribute__((ext_vector_type(4)));
typedef float f32x16 __attribute__((ext_vector_type(16)));

// lanes l and l ^ 32 hold the same query row
__device__ __forceinline__ float row2_max(float x) {
  const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
}
__device__ __forceinline__ float row2_sum(float x) {
  const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}

// Swizzled 16-byte chunk of (row, chunk) in an unpadded LDS tile of rows of D
// bf16, XORed by row so that (a) the same chunk of 16 consecutive rows (K reads)
// and (b) an aligned run of four chunks of four consecutive rows (V transpose
// reads of 32 dims) both cover all 64 banks once.
template <int D>
__device__ __forceinline__ int pf_chunk(int row, int chunk) {
  if constexpr (D == 128) return chunk ^ (((row & 3) << 2) | ((row >> 2) & 3));
  return chunk ^ ((((row >> 1) & 1) << 2) | ((row >> 2) & 3));
}

template <int D, bool ADD>
__global__ __launch_bounds__(256, 2) void prefill_kernel(PrefillArgs a) {
  constexpr int KC = D / 16;             // 16-dim chunks (score contraction)
  constexpr int DB = D / 32;             // 32-dim output blocks
  constexpr int CPR = D / 8;             // 16-byte chunks per K / V row
  constexpr int NI = kPfK * CPR / 256;   // DMA slots per thread per block and tensor
  __shared__ __attribute__((aligned(16))) uint16_t k_s[2][kPfK * D];
  __shared__ __attribute__((aligned(16))) uint16_t v_s[2][kPfK * D];

  // Workgroups are dealt to the eight XCDs round robin.  In launch order the
  // query blocks go from the longest causal range to the shortest, all heads of
  // all sequences at each, so every XCD gets the same work; with a multiple of
  // eight heads an XCD takes Hq / 8 consecutive heads of every sequence, which
  // share their K and V in its L2 as far as they are of one group: whole groups at
  // 32/8 heads (four heads an XCD), half a group at 32/4, whose K and V two XCDs
  // then read, and a quarter at 8/2.
  const uint32_t nqb = gridDim.x, NH = gridDim.y * gridDim.z;
  const uint32_t wg = blockIdx.x + nqb * (blockIdx.y + gridDim.y * blockIdx.z);
  const int qblk = (int)(nqb - 1 - wg / NH);
  const uint32_t hi = wg % NH;
  int h, b;
  if ((a.Hq & 7) == 0) {
    const uint32_t hpx = (uint32_t)a.Hq / 8, r = hi / 8;
    h = (int)((hi % 8) * hpx + r % hpx);
    b = (int)(r / hpx);
  } else {
    h = (int)(hi % (uint32_t)a.Hq);
    b = (int)(hi / (uint32_t)a.Hq);
  }
  const int tid = threadIdx.x;
  const int lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int r32 = lane & 31, g2 = lane >> 5;
  const int G = a.Hq / a.Hkv;
  const int Tb = (int)clamp_len(a.seq_lens, b, a.T);
  const int64_t qrow0 = ((int64_t)b * a.Hq + h) * a.T;
  const uint16_t* kh = a.k + (((int64_t)b * a.Hkv + h / G) * a.T) * D;
  const uint16_t* vh = a.v + (((int64_t)b * a.Hkv + h / G) * a.T) * D;
  // Softmax and gate in base-2 units (S' = S log2 e): exp(S~ - m) = 2^(S~' - m') and
  // sigmoid(beta (S - tau)) = 1 / (1 + 2^(-beta (S' - tau'))).  With c the raw
  // product q.k and s2 = log2(e) / sqrt(d): S' = s2 c, and the lane keeps
  // gs = s2 sigmoid = 1 / ((1 + e) / s2), so the gated score is c gs (no separate
  // scaling) and R = (sum of gs) / s2.
  constexpr float kLog2e = 1.4426950408889634f;
  const float s2 = kLog2e / sqrtf((float)D), is2 = 1.0f / s2;
  const float nbs = -a.beta * s2;
  const float C2 = a.C * kLog2e, C2is = C2 * is2;

  // the lane's row, and the B operands of the wavefront's queries (dims
  // 16 kc + 8 g2 .. + 7)
  const int wrow0 = qblk * kPfQ + 32 * w;
  const int t = wrow0 + r32, tq = min(t, a.T - 1);
  u32x4 qb[KC];
#pragma unroll
  for (int kc = 0; kc < KC; ++kc)
    qb[kc] = *reinterpret_cast<const u32x4*>(a.q + (qrow0 + tq) * D + 16 * kc + 8 * g2);
  const float btau2 = a.beta * a.tau[qrow0 + tq] * kLog2e;
  float m_i = 0.f;    // reference maximum; set by the first two units
  float l_i = 0.f;    // this lane's share of the row's weight sum
  float r_i = 0.f;    // this lane's share of the row's gate sum (times s2)
  f32x16 acc[DB];
#pragma unroll
  for (int db = 0; db < DB; ++db) acc[db] = f32x16{};
  // transpose reads of V: within a 16-lane group, lane provides key (lane & 15) / 4
  // and dims 4 (lane & 3) .. + 3 and receives four keys of dim lane & 15; groups
  // 0, 1 take keys 0..3 and groups 2, 3 keys 4..7 of a 32-dim block's halves
  const int vt_row = 4 * g2 + ((lane & 15) >> 2);
  const int vt_c = 2 * ((lane >> 4) & 1) + ((lane & 3) >> 1), vt_half = 4 * (lane & 1);

  // Key blocks of the workgroup, and 32-key units of this wavefront.  The
  // wavefront's last unit holds its diagonal (or the sequence's end) and is the
  // only one that needs a mask; the units after it, up to the workgroup's last
  // block, it skips.
  const int last_row = min(qblk * kPfQ + kPfQ, Tb) - 1;
  const int nkb = last_row >= 0 ? last_row / kPfK + 1 : 0;
  const int nu = wrow0 < Tb ? (min(wrow0 + 32, Tb) - 1) / 32 + 1 : 0;

  // DMA: LDS slot u = 256 j + tid (16 bytes, in order) of a block holds row
  // u / CPR, physical chunk u % CPR, i.e. the global chunk that the swizzle maps
  // there.  Slot j of a thread is row RPJ j + tid / CPR, and its swizzle term
  // (row bits 0 .. 3) does not depend on j, so the thread's byte offsets
  // within a block are goff + 4096 j; the block's base is wave-uniform.
  constexpr int RPJ = 256 / CPR;                     // rows per slot index
  static_assert(RPJ % 16 == 0, "the swizzle takes row bits 0 .. 3");
  const int grow0 = tid / CPR;
  const uint32_t goff = (uint32_t)(grow0 * D + 8 * pf_chunk<D>(grow0, tid % CPR)) * 2u;
  auto dma = [&](const uint16_t* src, uint16_t (*tile)[kPfK * D], int kb) {
    const char* base = reinterpret_cast<const char*>(src + (int64_t)kb * kPfK * D);
    uint16_t* dst = tile[kb & 1] + 8 * 64 * w;
    if ((kb + 1) * kPfK <= Tb) {
#pragma unroll
      for (int j = 0; j < NI; ++j)
        __builtin_amdgcn_global_load_lds((const void*)(base + goff + 4096 * j),
                                         (__attribute__((address_space(3))) void*)(dst + 8 * 256 * j),
                                         16, 0, 0);
    } else {          // rows past the sequence read its last row: whatever the cache holds
                      // there, NaN too, would reach p.V (with weight 0)
#pragma unroll
      for (int j = 0; j < NI; ++j) {
        const int row = RPJ * j + grow0;
        const uint32_t off = goff + 4096u * j -
                             (uint32_t)(row - (min(kb * kPfK + row, Tb - 1) - kb * kPfK)) * (2u * D);
        __builtin_amdgcn_global_load_lds((const void*)(base + off),
                                         (__attribute__((address_space(3))) void*)(dst + 8 * 256 * j),
                                         16, 0, 0);
      }
    }
  };

  // LDS element offsets of this lane's K operand (key row r32 of a 32-key half,
  // chunk 2 kc + g2) and V operand reads (16-key chunk c of a half); 16 and 32 rows
  // further the swizzle is the same
  auto read_k = [&](const uint16_t* kt, int kc) {
    return *reinterpret_cast<const u32x4*>(&kt[r32 * D + 8 * pf_chunk<D>(r32, 2 * kc + g2)]);
  };
  auto v_off = [&](int c, int db, int hi8) {
    const int row = vt_row + 8 * hi8;
    return (16 * c + row) * D + 8 * pf_chunk<D>(row, 4 * db + vt_c) + vt_half;
  };
  auto read_v = [&](const uint16_t* vt, int c, int db) {
    const i16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16(
        (__attribute__((address_space(3))) i16x4*)(&vt[v_off(c, db, 0)]));
    const i16x4 hi8 = __builtin_amdgcn_ds_read_tr16_b64_v4i16(
        (__attribute__((address_space(3))) i16x4*)(&vt[v_off(c, db, 1)]));
    const uint2 l2 = __builtin_bit_cast(uint2, lo), h2 = __builtin_bit_cast(uint2, hi8);
    return u32x4{l2.x, l2.y, h2.x, h2.y};
  };

  // arrive(kb), between units 2 kb and 2 kb + 1: this thread's DMAs are done; after
  // the barrier everyone's are (K of block kb + 1 and V of block kb are in LDS), and
  // everyone is done with the K of block kb and the V of block kb - 1, whose
  // buffers the next DMAs overwrite.  Every wavefront passes nkb + 1 barriers.
  auto arrive = [&](int kb) {
    __builtin_amdgcn_s_waitcnt(0);
    __syncthreads();
    if (kb + 2 < nkb) dma(kh, k_s, kb + 2);
    if (kb + 1 < nkb) dma(vh, v_s, kb + 1);
  };

  // One unit of 32 keys, its raw scores in s.  Its vector work is the gate and mask
  // (16 scores a lane), then the weights; the matrix work beside it is the previous
  // unit's NM p.V MFMAs (V half vt), all before the reference maximum may move, and
  // the NS score MFMAs of the next unit (K half kt), left in sn: NS1 of them beside
  // the gates, the rest beside the weights, so that both stretches carry their
  // share.  LDS operands are read LA MFMAs ahead.  MASKED: the wavefront's last
  // unit (keys past a row, keys past the sequence's end, and the row's own key,
  // which is not gated), with no next unit.  In every earlier unit each key precedes
  // every row of the wavefront.  Rows at or past the sequence's end compute on
  // regardless and are cleared when stored.
  constexpr int NS = KC, NM = 2 * DB, NS1 = 3 * NS / 8, LA = 3;
  constexpr int GS = 10, G0 = 2, CS = 5;   // gate steps, the first with MFMAs, weight steps
  u32x4 pw[2] = {u32x4{0, 0, 0, 0}, u32x4{0, 0, 0, 0}};   // the previous unit's weights (bf16 pairs)
  auto pv = [&](int n, const u32x4& va) {
    acc[n % DB] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, va),
                                                           __builtin_bit_cast(bf16x8, pw[n / DB]), acc[n % DB],
                                                           0, 0, 0);
  };
  auto score = [&](f32x16& c, int kc, const u32x4& ka) {
    c = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, ka),
                                                 __builtin_bit_cast(bf16x8, qb[kc]), c, 0, 0, 0);
  };
  auto unit = [&](int u, f32x16& s, f32x16& sn, const uint16_t* vt, const uint16_t* kt, auto masked_tag) {
    constexpr bool MASKED = decltype(masked_tag)::value;
    constexpr int NE = MASKED ? NM : NM + NS1;         // MFMAs beside the gates
    if constexpr (!MASKED) sn = f32x16{};
    u32x4 op[4];                                       // operands in flight
    auto rd = [&](int x) {                             // operand of MFMA x: p.V, then scores
      if (x < NM) op[x & 3] = read_v(vt, x / DB, x % DB);
      else if (!MASKED && x < NM + NS) op[x & 3] = read_k(kt, x - NM);
    };
    // gate, mask, gated score minus the reference maximum (base-2 units), two scores
    // a step, the three stages of a score one step apart so that no step waits for
    // its own transcendentals
    float y[16], e[4], gs[4], mx = kNegInf;
    float ru = 0.f, lu = 0.f;            // the unit's own sums (short chains: less rounding)
    const float nm = ADD ? -(C2 + m_i) : -m_i;
#pragma unroll
    for (int x = 0; x < LA; ++x) rd(x);
#pragma unroll
    for (int st = 0; st < GS; ++st) {
#pragma unroll
      for (int x = 0; x < NE; ++x)
        if (G0 + x * (GS - G0) / NE == st) {
          if (x < NM) pv(x, op[x & 3]); else score(sn, x - NM, op[x & 3]);
          rd(x + LA);
        }
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        if (st < 8) e[2 * (st & 1) + i] = __builtin_amdgcn_exp2f(fmaf(nbs, s[2 * st + i], btau2));
        if (st >= 1 && st < 9) {
          const int o = 2 * ((st - 1) & 1) + i;
          gs[o] = __builtin_amdgcn_rcpf(fmaf(e[o], is2, is2));
        }
      }
      if (st >= 2) {
        const int j0 = 2 * (st - 2);
        float gr[2];
#pragma unroll
        for (int i = 0; i < 2; ++i) {
          const int j = j0 + i;
          const float cv = s[j], gj = gs[j & 3];
          float x = ADD ? fmaf(C2is, gj, fmaf(cv, s2, nm)) : fmaf(cv, gj, nm);
          if constexpr (MASKED) {
            const int sk = u * 32 + 8 * (j >> 2) + 4 * g2 + (j & 3);
            const bool valid = sk <= t && t < Tb;
            gr[i] = valid ? gj : 0.f;
            if (sk == t) x = fmaf(cv, s2, -m_i);
            x = valid ? x : kNegInf;
          } else {
            gr[i] = gj;
          }
          y[j] = x;
        }
        ru = st == 2 ? gr[0] + gr[1] : ru + (gr[0] + gr[1]);
        mx = fmaxf(fmaxf(mx, y[j0]), y[j0 + 1]);
        // (the sums taken here: their adds are otherwise moved past the unit, and
        // the values they add stay in registers)
        asm volatile("" : "+v"(ru), "+v"(mx));
      }
      __builtin_amdgcn_sched_barrier(0);
    }
    r_i += ru;
    // The reference maximum is that of the first two units (64 keys) and afterwards
    // moves only when some row's maximum exceeds it by more than 8 (a wavefront-wide
    // decision): weights stay below 2^8, and the accumulators are rescaled only then.
    // (A row's largest weight is exact in bf16 when it is the reference.  With the
    // first unit's maximum alone that was rarer: output error against 64 bits at 16K
    // tokens, d = 128: 2.168e-3 with one unit, 2.148e-3 with two; 2000 tokens, d = 64:
    // 2.118e-3, 2.074e-3; the time is the same.)
    if (u <= 1 || __ballot(mx > 8.0f) != 0ull) {
      const float rm = row2_max(mx);
      const float dm = rm == kNegInf ? 0.f : (u == 0 ? rm : fmaxf(rm, 0.f));
      // (the first unit's move scales nothing: the sums are zero, and 2^-dm overflows
      // where the row's scores are below -128)
      const float alpha = u == 0 ? 1.0f : __builtin_amdgcn_exp2f(-dm);
      m_i += dm;
      l_i *= alpha;
#pragma unroll
      for (int db = 0; db < DB; ++db) acc[db] *= alpha;
#pragma unroll
      for (int j = 0; j < 16; ++j) y[j] -= dm;
    }
    // weights, four a step: the B operands of chunk c (keys 16 c + 4 g2 + j and
    // 16 c + 8 + 4 g2 + j, j < 4, on both operands of O^T += V^T P^T)
    float p[8];
#pragma unroll
    for (int st = 0; st < CS; ++st) {
      if constexpr (!MASKED) {
#pragma unroll
        for (int x = NE; x < NM + NS; ++x)
          if ((x - NE) * CS / (NM + NS - NE) == st) {
            score(sn, x - NM, op[x & 3]);
            rd(x + LA);
          }
      }
      if (st >= 1) {
        const int o = 4 * ((st - 1) & 1), j = st - 1;
        const float l4 = (p[o] + p[o + 1]) + (p[o + 2] + p[o + 3]);
        lu = st == 1 ? l4 : lu + l4;
        pw[j >> 1][2 * (j & 1)] = pack_bf16x2(p[o], p[o + 1]);
        pw[j >> 1][2 * (j & 1) + 1] = pack_bf16x2(p[o + 2], p[o + 3]);
        asm volatile("" : "+v"(lu));
      }
      if (st < 4) {
#pragma unroll
        for (int i = 0; i < 4; ++i) p[4 * (st & 1) + i] = __builtin_amdgcn_exp2f(y[4 * st + i]);
      }
      __builtin_amdgcn_sched_barrier(0);
    }
    l_i += lu;
  };

  if (nkb > 0) {
    constexpr int HALF = 32 * D;                       // elements of half a tile
    // the "previous unit" of unit 0 has zero weights: its V must be finite
    for (int i = tid; i < HALF / 8; i += 256) *reinterpret_cast<u32x4*>(&v_s[1][HALF + 8 * i]) = u32x4{0, 0, 0, 0};
    dma(kh, k_s, 0);
    if (nkb > 1) dma(kh, k_s, 1);
    dma(vh, v_s, 0);
    __builtin_amdgcn_s_waitcnt(0);
    __syncthreads();
    constexpr std::integral_constant<bool, false> plain{};
    constexpr std::integral_constant<bool, true> masked{};
    int kb = 0;
    if (nu > 0) {
      f32x16 s0 = f32x16{}, s1 = f32x16{};
#pragma unroll
      for (int kc = 0; kc < KC; ++kc) score(s0, kc, read_k(k_s[0], kc));
      // unit 2 k: p.V of V block k - 1's second half, scores of K block k's second half;
      // unit 2 k + 1: V block k's first half, K block k + 1's first half
      int u = 0;
      for (; u + 4 < nu; u += 4) {
        unit(u, s0, s1, v_s[1] + HALF, k_s[0] + HALF, plain);
        arrive(u >> 1);
        unit(u + 1, s1, s0, v_s[0], k_s[1], plain);
        unit(u + 2, s0, s1, v_s[0] + HALF, k_s[1] + HALF, plain);
        arrive((u >> 1) + 1);
        unit(u + 3, s1, s0, v_s[1], k_s[0], plain);
      }
      for (; u < nu - 1; ++u) {                        // the last three at most
        const int par = (u >> 1) & 1;
        unit(u, s0, s1, (u & 1) ? v_s[par] : v_s[par ^ 1] + HALF,
             (u & 1) ? k_s[par ^ 1] : k_s[par] + HALF, plain);
        if ((u & 1) == 0) arrive(u >> 1);
        s0 = s1;
      }
      kb = u >> 1;
      unit(u, s0, s1, (u & 1) ? v_s[kb & 1] : v_s[(kb & 1) ^ 1] + HALF, nullptr, masked);
      if ((u & 1) == 0) arrive(kb);
      const uint16_t* vt = v_s[kb & 1] + (u & 1) * HALF;
#pragma unroll
      for (int x = 0; x < NM; ++x) pv(x, read_v(vt, x / DB, x % DB));
      ++kb;
    }
    for (; kb < nkb; ++kb) arrive(kb);
  }
  // lane holds O[t][32 db + 8 (i / 4) + 4 g2 + i % 4]; rows at or past the
  // sequence's end are cleared
  const float ls = row2_sum(l_i);
  const float rs = row2_sum(r_i) * is2;
  if (t < a.T) {
    const bool row_ok = t < Tb && ls > 0.f;
    const float inv = row_ok ? 1.0f / ls : 0.f;
#pragma unroll
    for (int db = 0; db < DB; ++db) {
#pragma unroll
      for (int i = 0; i < 16; i += 4) {
        const uint32_t lo = row_ok ? pack_bf16x2(acc[db][i] * inv, acc[db][i + 1] * inv) : 0u;
        const uint32_t hi2 = row_ok ? pack_bf16x2(acc[db][i + 2] * inv, acc[db][i + 3] * inv) : 0u;
        *reinterpret_cast<uint2*>(a.out + (qrow0 + t) * D + 32 * db + 2 * i + 4 * g2) = make_uint2(lo, hi2);
      }
    }
    if (g2 == 0) {
      a.R[qrow0 + t] = t < Tb ? rs : 0.f;
      a.L[qrow0 + t] = row_ok ? (m_i + __log2f(ls)) * 0.6931471805599453f : kNegInf;
    }
  }
}

}  // namespace

hipError_t launch_prefill(const eta_prefill_desc_t& pd, const void* q, const void* k, const void* v,
                          const float* tau, const int32_t* seq_lens, void* out, float* R, float* L,
                          hipStream_t stream, LaunchHook hook) {
  PrefillArgs pa{reinterpret_cast<const uint16_t*>(q), reinterpret_cast<const uint16_t*>(k),
                 reinterpret_cast<const uint16_t*>(v), tau, seq_lens,
                 reinterpret_cast<uint16_t*>(out), R, L, pd.num_q_heads, pd.num_kv_heads,
                 pd.capacity_tokens, pd.beta, pd.C};
  dim3 grid((pd.capacity_tokens + kPfQ - 1) / kPfQ, pd.num_q_heads, pd.batch);
  return with_hook(hook, ETA_KERNEL_PREFILL, stream, [&] {
    if (pd.additive) {
      if (pd.head_dim == 64) hipLaunchKernelGGL((prefill_kernel<64, true>), grid, dim3(256), 0, stream, pa);
      if (pd.head_dim == 128) hipLaunchKernelGGL((prefill_kernel<128, true>), grid, dim3(256), 0, stream, pa);
    } else {
      if (pd.head_dim == 64) hipLaunchKernelGGL((prefill_kernel<64, false>), grid, dim3(256), 0, stream, pa);
      if (pd.head_dim == 128) hipLaunchKernelGGL((prefill_kernel<128, false>), grid, dim3(256), 0, stream, pa);
    }
  });
}

}  // namespace eta
