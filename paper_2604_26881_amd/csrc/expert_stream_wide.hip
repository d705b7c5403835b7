// Weight-streaming grouped GEMM for expert blocks with up to a few dozen rows per expert on average: the
// wide sibling of expert_stream_lds.hip (which serves batches of a few rows per expert).
//
//   gate/up : h[r, n]  = silu(<A[r,:], Wg[e][n,:]>) * <A[r,:], Wu[e][n,:]>
//   down    : Yp[r, n] = <A[r,:], Wd[e][n,:]>
//
// What bounds it: the weights, read once from HBM.  As there, a wave owns its output columns and a private
// ring of LDS stages, and there is no barrier; here it owns 64 weight rows (gate/up: 32 gate rows and the
// matching 32 up rows; down: 64 rows) and up to three blocks of 32 token rows, multiplied with MFMA 32x32x16.
// Every staged byte is then read from LDS exactly once, the copies of token rows (which come from L2 and
// share its path to LDS with the weights) are at most 1.5 times those of the weights, and an expert takes one
// pass over its weights up to 96 rows.
// (That is the coarse form; launches of few waves take 32 weight rows per wave, see launch_wide_any.)
//
// Work decomposition.  A pass is up to 96 rows of one expert; an item is one pass by 128 weight rows, one
// workgroup of two waves that share nothing but the item.  The number of passes depends on expert_offsets:
// every wave forms the prefix of the passes over the experts in registers and finds its item, so the hardware
// dispatcher balances the items and workgroups past the last item leave at once.  Items are ordered by expert,
// then column, then pass: the passes of a hot expert are neighbours and read the same weights at the same
// time.  Workgroup b runs on XCD b mod 8; the XCDs take runs of 8 consecutive items in turn, so an expert's
// token rows reach two or three L2s instead of all eight and the items of a hot expert are spread over the
// chip (one eighth of the items in one piece per XCD: 142 us instead of 135 on a batch of 301 tokens whose hot
// expert holds 298 rows).
//
// Measured, 60 experts, H 2048, I 1408, gate/up + down in us, against the kernels that served these sizes
// before (32-row passes streamed on all XCDs up to 26 rows per expert, then MFMA tiles):
//   13 rows per expert: 125 + 66 -> 120 + 61;  20: 133 + 72 -> 122 + 64;  26: 150 + 80 -> 125 + 66;
//   20 with a hot expert of 298 rows: 161 + 84 -> 135 + 73.
// 128 experts of 19 rows, H 1024, I 768: 86 + 47 -> 72 + 40.  The 692 MB of gate/up weights in 122 us are
// 5.7 TB/s.  Beyond about 32 rows per expert the copies of token rows cost more than the barrier of the MFMA
// tiles (34 rows: 134 + 72 here, 137 + 72 there; 40 rows: 141 + 76 and 138 + 73).
#include "common.h"
#include <algorithm>

namespace moe {

namespace {

constexpr int WIDE_EMAX = 256;      // experts of a block: four per lane
// A wave's weight rows and its ring (the choice: launch_wide_any).  COARSE: 64 rows, 40 KB: four waves fill the 160 KB of a
// CU.  FINE: 32 rows in the same ring.  FINEST: 32 rows in 24 KB: six waves fill a CU.
enum WideForm { COARSE, FINE, FINEST };
constexpr int wide_blocks(WideForm f) { return f == COARSE ? 2 : 1; }          // of 32 weight rows
constexpr int wide_ring(WideForm f) { return (f == FINEST ? 24 : 40) * 1024; }
constexpr int wide_rows(WideForm f) { return f == FINEST ? 64 : 96; }          // token rows per pass: two stages of them fit the ring
constexpr int wide_waves(WideForm f) { return f == COARSE ? 2 : 1; }           // waves (column blocks) per workgroup
constexpr int WIDE_RUN = 8;         // consecutive items of one XCD (4 ... 64 measured the same within 2 %)

template <int J, int NS, int NI, class F>
__device__ __forceinline__ void drain(F&& step) {
  if constexpr (J < NS) {
    wait_copies_but<(NS - 1 - J) * NI>();
    step();
    drain<J + 1, NS, NI>(step);
  }
}

// Where the rows of a pass come from and go: token rows A (through gather, if any), output C, elements between weight rows.
struct WideRows { const bf16_t* A; const int32_t* gather; bf16_t* C; int ldw; };

// One pass: TB token blocks (rows m0 .. of the expert's rows [rb, rb + Me)) by the weight rows at W0, W1: WB = 2: 32 at each;
// WB = 1: 16 at each (gate/up: the gate rows, then the up rows, in one MFMA block).  A product does not depend on its
// place in a block, so both give the same bits.
template <WideForm FORM, int TB, bool GATEUP>
__device__ __forceinline__ void wide_pass(const GemmArgs& a, const WideRows& r, unsigned char* ring, int rb, int Me, int m0, int mend,
                                          int n0, int rot, const unsigned char* W0, const unsigned char* W1) {
  constexpr int WB = wide_blocks(FORM);
  constexpr int STAGE = (WB + TB) * 4096;  // 32 * WB weight rows, then TB x 32 token rows, 128 bytes each
  constexpr int NS = wide_ring(FORM) / STAGE;   // COARSE 3, 2, 2; FINE 5, 3, 2; FINEST 3, 2
  constexpr int NI = (WB + TB) * 4;        // 1 KB copies per stage
  constexpr int NW0 = 2 * WB;              // of which the first are the rows at W0, as many those at W1
  static_assert(NS >= 2 && (NS - 1) * NI < 64, "the wait counter holds 6 bits");
  const int lane = threadIdx.x & 63;
  const int N = a.N, Kdim = a.Kdim, nk = Kdim / 64;
  const unsigned char* Ab = reinterpret_cast<const unsigned char*>(r.A);
  const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) unsigned char*)ring;
  // copies: lane -> row lane/8 of an 8-row group, slot lane%8 holding chunk slot xor row%8
  const int crow = lane >> 3, cchunk = (lane & 7) ^ crow;
  uint32_t coffW[NW0], coffX[TB * 4];
#pragma unroll
  for (int i = 0; i < NW0; ++i) coffW[i] = (uint32_t)(i * 8 + crow) * (uint32_t)r.ldw * 2u + (uint32_t)cchunk * 16u;
#pragma unroll
  for (int i = 0; i < TB * 4; ++i) {
    const int m = min(m0 + i * 8 + crow, Me - 1);   // rows past the end repeat the last row
    const int arow = r.gather ? r.gather[rb + m] / a.gather_div : rb + m;
    coffX[i] = (uint32_t)arow * (uint32_t)Kdim * 2u + (uint32_t)cchunk * 16u;
  }
  const int r32 = lane & 31, half = lane >> 5, swz = lane & 7;
  f32x16 acc[WB][TB];
#pragma unroll
  for (int b = 0; b < WB; ++b)
#pragma unroll
    for (int t = 0; t < TB; ++t)
#pragma unroll
      for (int i = 0; i < 16; ++i) acc[b][t][i] = 0.0f;

  auto kbyte = [&](int s) -> size_t { return (size_t)(s + rot >= nk ? s + rot - nk : s + rot) * 128; };
  auto request1 = [&](size_t kb, int slot, int i) {   // copy i of the stage of the K step at byte kb of the rows
    const uint32_t l = lds0 + (uint32_t)slot * STAGE + (uint32_t)i * 1024u;
    if (i < NW0) copy_to_lds_16(W0 + kb, coffW[i], l, true);
    else if (i < 2 * NW0) copy_to_lds_16(W1 + kb, coffW[i - NW0], l, true);
    else copy_to_lds_16(Ab + kb, coffX[i - 2 * NW0], l);
  };
  // Multiply the stage in `slot`: all operands go to registers first (the empty asm makes the compiler wait for
  // them), so the slot is free and takes, request by request between the MFMAs, the stage NS steps ahead.
  auto consume = [&](int slot, bool more, size_t kb) {
    const unsigned char* st = ring + slot * STAGE + r32 * 128;
    u32x4 w[WB][4], x[TB][4];
#pragma unroll
    for (int kk = 0; kk < 4; ++kk) {
      const int c = ((2 * kk + half) ^ swz) << 4;
#pragma unroll
      for (int b = 0; b < WB; ++b) w[b][kk] = *reinterpret_cast<const u32x4*>(st + b * 4096 + c);
#pragma unroll
      for (int t = 0; t < TB; ++t) x[t][kk] = *reinterpret_cast<const u32x4*>(st + (WB + t) * 4096 + c);
    }
#pragma unroll
    for (int kk = 0; kk < 4; ++kk) {
#pragma unroll
      for (int b = 0; b < WB; ++b) asm volatile("" : "+v"(w[b][kk]));
#pragma unroll
      for (int t = 0; t < TB; ++t) asm volatile("" : "+v"(x[t][kk]));
    }
#pragma unroll
    for (int j = 0; j < 4 * WB * TB; ++j) {
      const int kk = j / (WB * TB), b = j % WB, t = (j / WB) % TB;
      acc[b][t] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(as_bf16x8(w[b][kk]), as_bf16x8(x[t][kk]), acc[b][t], 0, 0, 0);
      if (more) {
#pragma unroll
        for (int i = 0; i < NI; ++i)
          if (i * 4 * WB * TB / NI == j) request1(kb, slot, i);
      }
      __builtin_amdgcn_sched_barrier(0x6);
    }
  };
  // (nk >= NS: shorter contractions go to the narrow kernel)
  for (int s = 0; s < NS; ++s) {
    const size_t kb = kbyte(s);
#pragma unroll
    for (int i = 0; i < NI; ++i) request1(kb, s, i);
  }
  int slot = 0;
  for (int s = 0; s + NS < nk; ++s) {
    wait_copies_but<(NS - 1) * NI>();   // step s has landed
    consume(slot, true, kbyte(s + NS));
    slot = slot + 1 == NS ? 0 : slot + 1;
  }
  drain<0, NS, NI>([&]() {
    consume(slot, false, 0);
    slot = slot + 1 == NS ? 0 : slot + 1;
  });
  // accumulator element i of block (b, t): weight row (output column) 8*(i/4) + 4*(lane/32) + i%4 of the block,
  // token row lane%32; lanes l and l+32 trade column groups, so each stores 16 bytes
#pragma unroll
  for (int t = 0; t < TB; ++t) {
    const int m = m0 + t * 32 + r32;
    if (m < mend) {
      bf16_t* out = r.C + (size_t)(rb + m) * N + n0;
#pragma unroll
      for (int b = 0; b < (GATEUP ? 1 : WB); ++b) {
#pragma unroll
        for (int q = 0; q < (GATEUP && WB == 1 ? 2 : 4); q += 2) {
          float v[8];
#pragma unroll
          for (int i = 0; i < 8; ++i) {
            const float g = acc[b][t][4 * q + i];
            v[i] = GATEUP ? __fdividef(g, 1.0f + __expf(-g)) * (WB == 1 ? acc[0][t][8 + i] : acc[WB - 1][t][4 * q + i]) : g;
          }
          uint32_t ox = pack_bf16x2(v[0], v[1]), oy = pack_bf16x2(v[2], v[3]);
          uint32_t oz = pack_bf16x2(v[4], v[5]), ow = pack_bf16x2(v[6], v[7]);
          trade_halves(ox, oz);
          trade_halves(oy, ow);
          *reinterpret_cast<u32x4*>(out + b * 32 + 8 * (q + half)) = u32x4{ox, oy, oz, ow};
        }
      }
    }
  }
}

// SHARED: a.n_shared more weight sets of N by Kdim ride along, each applied to all a.shared_rows tokens (the block call that
// hosts the shared experts); their items come first, for they have the most rows.
template <bool GATEUP, bool SHARED, WideForm FORM>
__global__ __launch_bounds__(64 * wide_waves(FORM)) void expert_stream_wide_kernel(GemmArgs a, int groups) {
  extern __shared__ __align__(16) unsigned char smem[];
  constexpr int WB = wide_blocks(FORM), ROWS = wide_rows(FORM);
  constexpr int NPER = (GATEUP ? 16 : 32) * WB;   // output columns of a wave
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int nsets = SHARED ? a.n_shared : 0;
  const int nexp = nsets + a.hi - a.lo;

  // passes of the experts (four per lane) and their exclusive prefix
  int eid[4], rb[4], me[4], np[4], sum = 0;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int e = lane * 4 + i;
    eid[i] = 0; rb[i] = 0; me[i] = 0; np[i] = 0;
    if (SHARED && e < nsets) {
      eid[i] = -1 - e;
      me[i] = a.shared_rows;
      np[i] = (me[i] + ROWS - 1) / ROWS;
    } else if (e < nexp) {
      eid[i] = a.ids ? a.ids[a.lo + e - nsets] : a.lo + e - nsets;
      rb[i] = a.offsets[eid[i]];
      me[i] = a.offsets[eid[i] + 1] - rb[i];
      np[i] = (max(me[i], 0) + ROWS - 1) / ROWS;
    }
    sum += np[i];
  }
  int incl = sum;
#pragma unroll
  for (int s = 1; s < 64; s <<= 1) {
    const int o = __shfl_up(incl, s, WAVE);
    if (lane >= s) incl += o;
  }
  const int items = __builtin_amdgcn_readlane(incl, 63) * groups;
  const int p = (int)(blockIdx.x >> 3);
  const int run = p / WIDE_RUN;
  const int item = (run * 8 + (int)(blockIdx.x & 7)) * WIDE_RUN + (p - run * WIDE_RUN);
  if (item >= items) return;
  // the expert of the item: in the last lane whose prefix is not beyond it
  int base = (incl - sum) * groups;
  const int src = 63 - __builtin_clzll(__ballot(base <= item));
  int le = eid[0], lrb = rb[0], lme = me[0], lnp = np[0];
#pragma unroll
  for (int i = 1; i < 4; ++i) {
    const int next = base + lnp * groups;
    if (item >= next) { base = next; le = eid[i]; lrb = rb[i]; lme = me[i]; lnp = np[i]; }
  }
  const int id = __builtin_amdgcn_readlane(le, src);
  const bool sh = SHARED && id < 0;
  const int eg = sh ? -1 - id : id;     // the expert, or the number of the shared set
  const int erb = __builtin_amdgcn_readlane(lrb, src);
  const int Me = __builtin_amdgcn_readlane(lme, src);
  const int passes = __builtin_amdgcn_readlane(lnp, src);
  const int rem = item - __builtin_amdgcn_readlane(base, src);
  const int group = passes > 1 ? rem / passes : rem;
  const int pass = rem - group * passes;

  const int N = a.N, Kdim = a.Kdim, nk = Kdim / 64;
  const int col = group * wide_waves(FORM) + wave;
  const int n0 = col * NPER;
  if (n0 >= N) return;
  // rows of the pass: the expert's 32-row blocks dealt evenly to its passes
  const int blocks = (Me + 31) >> 5;
  const int b0 = blocks * pass / passes, b1 = blocks * (pass + 1) / passes;
  // the walk over K starts at a step of its own (see expert_stream_lds.hip); it depends on the expert and the
  // column only, so results depend neither on the block cut nor on the passes
  const int rot = (int)(((unsigned)(WB == 1 ? col >> 1 : col) * 3u + (unsigned)eg * 5u) % (unsigned)nk);   // (32 or 64 columns)
  WideRows r{a.A, a.gather, a.C, Kdim};
  const bf16_t *B0 = a.B0 + (size_t)eg * N * Kdim, *B1 = GATEUP ? a.B1 + (size_t)eg * N * Kdim : nullptr;
  if (sh) {    // gate/up: every set reads the tokens; down: its own hidden rows
    r = WideRows{a.As + (GATEUP ? (size_t)0 : (size_t)eg * a.shared_rows * Kdim), nullptr, a.Cs + (size_t)eg * a.shared_rows * N, a.ldb_shared};
    B0 = a.Bs0 + (size_t)eg * a.shared_b_step;
    B1 = GATEUP ? a.Bs1 + (size_t)eg * a.shared_b_step : nullptr;
  }
  const unsigned char* W0 = reinterpret_cast<const unsigned char*>(B0 + (size_t)n0 * r.ldw);
  const unsigned char* W1 = GATEUP ? reinterpret_cast<const unsigned char*>(B1 + (size_t)n0 * r.ldw) : W0 + (size_t)(16 * WB) * r.ldw * 2;
  unsigned char* ring = smem + wave * wide_ring(FORM);
  const int m0 = b0 * 32, mend = min(b1 * 32, Me);
  switch (b1 - b0) {
    case 1: wide_pass<FORM, 1, GATEUP>(a, r, ring, erb, Me, m0, mend, n0, rot, W0, W1); break;
    case 2: wide_pass<FORM, 2, GATEUP>(a, r, ring, erb, Me, m0, mend, n0, rot, W0, W1); break;
    default: if constexpr (ROWS > 64) wide_pass<FORM, 3, GATEUP>(a, r, ring, erb, Me, m0, mend, n0, rot, W0, W1); break;
  }
}

template <bool GATEUP, bool SHARED, WideForm FORM>
int launch_wide(const GemmArgs& a, hipStream_t st) {
  auto kern = expert_stream_wide_kernel<GATEUP, SHARED, FORM>;
  constexpr int lds = wide_waves(FORM) * wide_ring(FORM), ROWS = wide_rows(FORM);
  const int nexp = a.hi - a.lo, nsets = SHARED ? a.n_shared : 0;
  if (a.offsets == nullptr || nexp + nsets > WIDE_EMAX || a.N % 64 != 0 || a.Kdim % 64 != 0 || a.Kdim < 5 * 64) return -2;   // (the deepest ring)
  const int per = wide_waves(FORM) * (GATEUP ? 16 : 32) * wide_blocks(FORM);
  const int groups = (a.N + per - 1) / per;
  // an upper bound of the passes: every expert's last pass may be partial
  const long passes = (long)a.rows_total / ROWS + std::min((long)nexp, (long)a.rows_total) +
                      (long)nsets * ((a.shared_rows + ROWS - 1) / ROWS);
  constexpr long runs = 8l * WIDE_RUN;
  const long grid = (passes * groups + runs - 1) / runs * runs;
  if (grid <= 0) return 0;
  static std::atomic<uint64_t> lds_raised{0};
  if (raise_lds_limit((const void*)kern, lds, lds_raised) != 0) return -4;
  hipLaunchKernelGGL(kern, dim3((unsigned)grid), dim3(64 * wide_waves(FORM)), lds, st, a, groups);
  return hipGetLastError() == hipSuccess ? 0 : -4;
}

// The forms give the same bits, so the choice may look at the call (a few experts of a layer cut into blocks).  By waves of 64
// weight rows, counting one pass per expert, on 256 CUs: up to 1.5 per CU a launch is bound by the latency of its few
// waves, and twice as many of half the rows are faster (4 of 16 experts, H 3072, I 2048, 16 rows, gate/up: 256 waves, 27.4
// -> 19.7 us; 352: 35.6 -> 34.5; 440: 22.0 -> 23.8); up to 2 every CU has one coarse workgroup at most; up to 3 some have
// two and the rest one, while the six finest waves that fit a CU come out even (15 of 60, H 2048, I 1408, 11 rows, gate/up:
// 660 waves, 37.5 -> 31.9 us; 768, H 1024: 21.7 -> 18.8; 880: 40.1 -> 41.9); beyond, the token rows, which the fine forms copy
// twice as often, cost more than that.
template <bool GATEUP>
int launch_wide_any(const GemmArgs& a, hipStream_t st) {
  if (a.n_shared > 0) return launch_wide<GATEUP, true, COARSE>(a, st);
  const long waves = std::min((long)(a.hi - a.lo), (long)a.rows_total) * (a.N / (GATEUP ? 32 : 64));
  if (waves <= 384) return launch_wide<GATEUP, false, FINE>(a, st);
  if (waves > 512 && waves <= 768) return launch_wide<GATEUP, false, FINEST>(a, st);
  return launch_wide<GATEUP, false, COARSE>(a, st);
}

}  // namespace

int launch_stream_wide_gateup(const GemmArgs& a, hipStream_t st) { return launch_wide_any<true>(a, st); }
int launch_stream_wide_down(const GemmArgs& a, hipStream_t st) { return launch_wide_any<false>(a, st); }

}  // namespace moe
