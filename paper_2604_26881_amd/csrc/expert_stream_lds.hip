// Weight-streaming grouped GEMM for expert blocks with FEW rows per expert, weights staged through
// LDS.  FaaSMoE Sec. 3: an expert block computes statelessly on the tokens it is handed; at decode
// sizes an expert sees a handful of rows, so the work is reading its weights once from HBM, and
// experts without rows return at once (only activated experts cost anything).
//
//   gate/up : h[r, n]  = silu(<A[r,:], Wg[e][n,:]>) * <A[r,:], Wu[e][n,:]>
//   down    : Yp[r, n] = <A[r,:], Wd[e][n,:]>
//
// Why LDS: the MFMA 16x16x32 operand layout gives a weight row to only four lanes, so loading the
// operand straight into registers asks memory for 16 rows x 64 bytes (or interleaved 16-byte
// pieces) per instruction.  Measured on a 1 GiB read of 4 KB rows, that request shape reaches
// 5.7-5.9 TB/s, whole 128-byte lines per row (8 lanes per row) reach 6.8 TB/s.  So the weights are
// copied global -> LDS with 8 lanes per row (one full line each, no registers in between) and the
// MFMA operands are read back from LDS in the layout the matrix core wants.
//
// One wave per workgroup, no barrier anywhere: a wave owns two 16-row weight blocks (gate/up: a
// gate block and the matching up block, so SwiGLU is formed in registers; down: two neighbouring
// blocks) and MT tiles of 16 token rows.  Per 64-wide K step it copies 2 x 16 x 128 bytes of
// weights and MT x 16 x 128 bytes of token rows into its own ring of NST LDS stages; NST-1 stages
// are in flight while one is multiplied.  Copies complete in issue order, so "all but the newest
// (NST-2) stages have landed" is a plain s_waitcnt vmcnt(n).  Token rows go through the same ring
// (they come from L2): a register load of them would sit in the same in-order queue behind the
// deep weight prefetch and drain it.  A row's eight 16-byte chunks are stored at slot = chunk xor
// row%8, which keeps the operand reads (16 rows, same chunk) off each other's banks.
// Several such workgroups share a CU (LDS decides how many), so the start-up of one overlaps the
// steady state of the others, and the hardware dispatcher balances the 16-row blocks dynamically.
// An expert with more rows than one pass covers (16 x MT) re-reads its weights once per pass; its
// passes are spread over up to eight workgroups, so that the hot expert of a skewed batch does not
// become one long chain.
#include "common.h"

namespace moe {

template <int MT, int NST>
struct StreamLdsShape {
  static constexpr int WBYTES = 2 * 16 * 128;   // two weight blocks, one K step
  static constexpr int XBYTES = MT * 16 * 128;  // token tiles, one K step
  static constexpr int STAGE = WBYTES + XBYTES;
  static constexpr int NI = 4 + 2 * MT;         // 1 KB copies per stage
  static constexpr int D = NST - 1;             // stages in flight
  static_assert(D >= 1 && D * NI < 64, "the wait counter holds 6 bits");
};

// SORT (gate/up of a layer with few pairs): the launch constructs the micro-batch as well.  A wave needs little of it: how
// many pairs chose its expert, how many a lower one, and which pairs its rows are.  Each reads that off the expert ids
// themselves with a ballot per 64 pairs (in the place of two dependent loads of the sorted arrays), and the workgroups of
// blockIdx.y == 0 write the arrays, and the row copies where asked for, for the launches that follow: the same stable
// counting sort as in permute.hip, by one wave.
// It saves a launch of 3-4 us and the gap before it, and costs every wave its look at the ids, also those of experts without
// rows: the rule beside sort_in_gateup draws the line.  A layer, us, sorted in a launch of its own -> here: H 64, 16 tokens,
// top 2 25.8 -> 22.7; 60 experts of H 2048, I 1408, top 4 at 1 token 46.4 -> 42.6, at 13 125.4 -> 122.9, at 30 (120 pairs) 182.2 ->
// 180.1; 256 of H 1024, I 256, top 8 at 8 tokens 39.6 -> 36.1, at 16 (128 pairs) 54.5 -> 52.9.  Beyond 128 pairs it turns everywhere: 160
// pairs of the 60 experts 194 -> 198, 180 of 64 experts of H 1536 114 -> 118, 1024 of the 256 96 -> 148.
constexpr int SORT_SPLIT = 16;   // waves that share the row copies of 64 pairs
__device__ __forceinline__ int pair_expert(const GemmArgs& a, int p) {   // -1 past the last pair
  return p < a.n_pairs ? min(max(a.sort_ids[p], 0), a.experts_layer - 1) : -1;   // (an id outside [0,E) stays in the tables)
}
__device__ __forceinline__ void sort_pairs(const GemmArgs& a, int* lds) {
  int* const s_total = lds;          // pairs of expert e
  int* const s_base = lds + 256;     // those in earlier chunks; then: first row of expert e for this chunk
  int* const s_row = lds + 512;
  const int lane = threadIdx.x, E = a.experts_layer, nbits = bits_for(E);
  const int chunks = (a.n_pairs + 63) / 64, split = a.sort_copy != nullptr ? SORT_SPLIT : 1;
  for (int item = blockIdx.x; item < chunks * split; item += gridDim.x) {
    const int c = item / split, part = item % split;
    for (int i = lane; i < 512; i += 64) lds[i] = 0;
    __syncthreads();
    for (int cc = 0; cc < chunks; ++cc) {
      const int e = pair_expert(a, cc * 64 + lane);
      const unsigned long long match = match_expert(max(e, 0), e >= 0, nbits);
      if (e >= 0 && (match & ((1ull << lane) - 1ull)) == 0ull) {   // one lane per expert
        s_total[e] += __popcll(match);
        if (cc < c) s_base[e] += __popcll(match);
      }
      __syncthreads();
    }
    int v[4], sum = 0;   // exclusive scan of the totals over experts, four experts per lane
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      v[i] = s_total[lane * 4 + i];   // (zero beyond E)
      sum += v[i];
    }
    int incl = sum;
#pragma unroll
    for (int s = 1; s < 64; s <<= 1) {
      const int o = __shfl_up(incl, s, WAVE);
      if (lane >= s) incl += o;
    }
    int base = incl - sum;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int e = lane * 4 + i;
      s_base[e] += base;
      if (item == 0 && e < E) a.sort_offsets[e] = base;
      base += v[i];
    }
    if (item == 0 && lane == 63) a.sort_offsets[E] = incl;
    __syncthreads();
    const int p = c * 64 + lane, own = pair_expert(a, p);
    const unsigned long long match = match_expert(max(own, 0), own >= 0, nbits);
    int row = -1;
    if (own >= 0) {
      row = s_base[own] + __popcll(match & ((1ull << lane) - 1ull));
      if (part == 0) {
        a.sort_rows[p] = row;
        a.sort_src[row] = p;
      }
    }
    s_row[lane] = row;
    __syncthreads();
    if (a.sort_copy != nullptr) {
      for (int i = part; i < 64; i += split) {
        const int to = s_row[i];
        if (to < 0) break;                      // pairs past the last sit at the end of the last chunk
        const u32x4* src = reinterpret_cast<const u32x4*>(a.A + (size_t)((c * 64 + i) / a.gather_div) * a.Kdim);
        u32x4* dst = reinterpret_cast<u32x4*>(a.sort_copy + (size_t)to * a.Kdim);
        for (int j = lane; j < a.Kdim / 8; j += 64) dst[j] = src[j];
      }
    }
    __syncthreads();
  }
}

template <int J, int D, int NI, class F>
__device__ __forceinline__ void stream_tail(F&& step) {
  if constexpr (J < D) {
    wait_copies_but<(D - 1 - J) * NI>();
    step(J);
    stream_tail<J + 1, D, NI>(step);
  }
}

// SHARED: the shared expert of a batch of a few tokens, riding along with the routed experts or (no experts) by itself.
// Of blockIdx.y the first a.n_shared are its own, and all of them take all tokens.  Gate/up: sets of N columns of its
// hidden layer (the last one may be narrower).  Down: its contraction is cut into a.shared_parts parts of whole K steps;
// with a.Cpart each is a set of its own and leaves fp32 partial sums there, which a later kernel adds in ascending order
// and rounds; without room for them there is one set (TURN) and one wave forms the parts one after another and adds them in
// that same order.  (With as many sets as parts and no a.Cpart every part is an output of its own, bf16 in a.Cs: the block call that hosts
// the shared experts.)
// The parts and the K starts depend on Is and the column alone, so the shared expert has the same bits alone, riding,
// beside any block cut, and whatever the workspace.
// With one token the routed experts and the shared expert each leave most of the chip idle in a launch of their own:
// H 2048, 4 of 60 experts of I 1408 and Is 5632, gate/up 14.8 + 16.3 us, down 8.3 + 13.3 (tiles with K cut in 8, and their
// sum); together 19.2 and 11.3.  By itself (beside several blocks or on a second stream), with its sum and gate logits,
// against those tiles: 1 token 32 -> 21 us, 32 tokens 32 -> 24; H 1024, Is 4032 42 -> 14.  From 17 tokens on a riding shared expert is read by two passes; up to 32 tokens that
// still beats launches of their own on one stream.
template <int MT, bool GATEUP, int NST, bool SHARED, bool TURN, bool SORT>
__global__ __launch_bounds__(64) void expert_stream_lds_kernel(GemmArgs a) {
  using S = StreamLdsShape<MT, NST>;
  extern __shared__ __align__(16) unsigned char smem[];
  constexpr int NPER = GATEUP ? 16 : 32;   // output columns of one item (two 16-row weight blocks)

  static_assert(!SORT || GATEUP, "the micro-batch is constructed beside the first kernel of the layer");
  const int lane = threadIdx.x;
  if (SORT && blockIdx.y == 0) {
    if (blockIdx.z == 0) sort_pairs(a, reinterpret_cast<int*>(smem));
    return;
  }
  const int by = (int)blockIdx.y - (SORT ? 1 : 0);
  const bool sh = SHARED && by < a.n_shared;   // eg: the shared set, otherwise the expert id
  const int y = by - (SHARED && !sh ? a.n_shared : 0);
  const int eg = sh ? y : a.offsets ? (a.ids ? a.ids[a.lo + y] : a.lo + y) : 0;
  // SORT: pairs [m0, m0 + pass_rows) of this expert, in order, into s_pair; the pairs of lower experts and of this one
  int* const s_pair = reinterpret_cast<int*>(smem);   // (the ring is free whenever this is called)
  auto own_pairs = [&](int first, int& lower, int& mine) {
    lower = mine = 0;
    for (int p0 = 0; p0 < a.n_pairs; p0 += 128) {   // two requests at a time
      int e[2];
#pragma unroll
      for (int u = 0; u < 2; ++u) e[u] = pair_expert(a, p0 + u * 64 + lane);
#pragma unroll
      for (int u = 0; u < 2; ++u) {
        const unsigned long long match = __ballot(e[u] == eg);
        const int rank = mine + __popcll(match & ((1ull << lane) - 1ull)) - first;
        if (e[u] == eg && rank >= 0 && rank < 16 * MT) s_pair[rank] = p0 + u * 64 + lane;
        mine += __popcll(match);
        lower += __popcll(__ballot(e[u] >= 0 && e[u] < eg));
      }
    }
    __syncthreads();   // (one wave: orders the writes above before the reads of other lanes)
  };
  int rb = 0, Me = 0;
  if (SORT && !sh) {
    own_pairs((int)blockIdx.z * 16 * MT, rb, Me);
  } else {
    rb = a.offsets && !sh ? a.offsets[eg] : 0;
    Me = (sh ? a.shared_rows : a.offsets ? a.offsets[eg + 1] : a.rows_fixed) - rb;
  }
  // An expert with more rows than one pass covers takes further passes over its weights.  They are dealt
  // round-robin to the gridDim.z workgroups of this (expert, column block): workgroups without a pass leave
  // at once (they cost nothing measurable), and a hot expert of a skewed batch no longer runs all its passes
  // one after another in one wave while the rest of the chip has finished.
  const int pass_rows = 16 * MT;
  if (Me <= (int)blockIdx.z * pass_rows) return;

  const int N = a.N;
  constexpr bool CUT = SHARED && !GATEUP;                      // a shared set's contraction comes in parts
  const int Kdim = CUT && sh ? a.ldb_shared : a.Kdim;          // elements between consecutive weight (and token) rows
  static_assert(!TURN || CUT, "parts of the shared contraction");
  const int part0 = CUT && sh && !TURN ? eg : 0;               // the parts this wave forms
  const int part1 = TURN ? a.shared_parts : part0 + 1;
  int nk = Kdim / 64;                                          // K steps of a part, and the byte where it begins
  size_t kofs = 0;
  // The walk over K starts at step `rot` and wraps around.  Thousands of these waves start within a
  // few microseconds of each other; if all began at K step 0 their requests of one moment would sit
  // at the same offset inside the weight rows, which for rows of a power-of-two length (4 KB at
  // K = 2048) lands them in the same memory channels (measured on the decode batch: gate/up 134 us
  // with a common start, 121 us with staggered starts; the 2816-byte rows of the down projection
  // show no difference).  rot depends on the expert (or the part) and the column block only, so results
  // do not depend on the block cut.
  auto start = [&](unsigned column, unsigned set) { return (int)((column * 3u + set * 5u) % (unsigned)nk); };
  // this wave's output columns: rows [n0, n0+16) of both branches (gate/up) or rows [n0, n0+32) (down)
  const int n0 = (int)blockIdx.x * NPER;
  if (n0 >= N || (sh && GATEUP && eg * N + n0 >= a.ldb_shared)) return;
  int rot = sh && GATEUP ? start((unsigned)(eg * N + n0) / NPER, 0u) : start(blockIdx.x, (unsigned)eg);
  const size_t wrow = sh && !GATEUP ? (size_t)n0 : (size_t)eg * N + n0;   // first weight row
  const unsigned char* W0 = reinterpret_cast<const unsigned char*>((sh ? a.Bs0 : a.B0) + wrow * Kdim);
  const unsigned char* W1 = GATEUP ? reinterpret_cast<const unsigned char*>((sh ? a.Bs1 : a.B1) + wrow * Kdim)
                                   : W0 + (size_t)16 * Kdim * 2;
  const unsigned char* Ab = reinterpret_cast<const unsigned char*>(sh ? a.As : a.A);
  const bool gathered = a.gather != nullptr && !sh;
  // gate/up: the shared hidden rows are ldb_shared wide, set eg owns columns [eg*N, (eg+1)*N) of them
  bf16_t* const Cb = sh ? a.Cs + (GATEUP ? (size_t)eg * N : (size_t)eg * a.shared_rows * N) : a.C;
  const int ldc = sh && GATEUP ? a.ldb_shared : N;

  const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) unsigned char*)smem;
  // copies: lane -> row lane/8 of an 8-row group, slot lane%8 holding chunk slot xor row%8
  const int crow = lane >> 3;
  const int cchunk = (lane & 7) ^ crow;
  uint32_t coffW[2];
#pragma unroll
  for (int i = 0; i < 2; ++i) coffW[i] = (uint32_t)(i * 8 + crow) * (uint32_t)Kdim * 2u + (uint32_t)cchunk * 16u;
  // operand reads: lane -> row lane%16, chunk 4*j + lane/16 for the j-th MFMA of the K step
  const int r16 = lane & 15, q = lane >> 4;
  const int frag_off = r16 * 128;
  const int swz = r16 & 7;

  for (int m0 = (int)blockIdx.z * pass_rows; m0 < Me; m0 += pass_rows * (int)gridDim.z) {
    if (SORT && !sh && m0 != (int)blockIdx.z * pass_rows) {
      int lower, mine;
      own_pairs(m0, lower, mine);
    }
    uint32_t coffX[MT][2];
#pragma unroll
    for (int mt = 0; mt < MT; ++mt)
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        const int m = min(m0 + mt * 16 + i * 8 + crow, Me - 1);   // rows past the end repeat the last row
        const int arow = SORT && !sh ? s_pair[m - m0] / a.gather_div : gathered ? a.gather[rb + m] / a.gather_div : rb + m;
        coffX[mt][i] = (uint32_t)arow * (uint32_t)Kdim * 2u + (uint32_t)cchunk * 16u;
      }
    // s_pair lies in ring slot 0, and the first copies into that slot, of weights, do not depend on what is read from it here
    if (SORT && !sh) wait_lds_reads();

    f32x4 acc0[MT], acc1[MT];

    // K step s into ring slot `slot`: the weights with the read-once hint, the token rows without
    auto issue = [&](int s, int slot) {
      const uint32_t l = lds0 + (uint32_t)slot * S::STAGE;
      const size_t kb = kofs + (size_t)(s + rot >= nk ? s + rot - nk : s + rot) * 128;
      copy_to_lds_16(W0 + kb, coffW[0], l, true);
      copy_to_lds_16(W0 + kb, coffW[1], l + 1024u, true);
      copy_to_lds_16(W1 + kb, coffW[0], l + 2048u, true);
      copy_to_lds_16(W1 + kb, coffW[1], l + 3072u, true);
#pragma unroll
      for (int mt = 0; mt < MT; ++mt) {
        copy_to_lds_16(Ab + kb, coffX[mt][0], l + (uint32_t)S::WBYTES + (uint32_t)mt * 2048u);
        copy_to_lds_16(Ab + kb, coffX[mt][1], l + (uint32_t)S::WBYTES + (uint32_t)mt * 2048u + 1024u);
      }
    };
    // accumulator element j of tile mt: weight row (output column) 4*(lane/16) + j of the block,
    // token row lane%16
    auto store = [&]() {
#pragma unroll
      for (int mt = 0; mt < MT; ++mt) {
        const int m = m0 + r16 + mt * 16;
        if (m < Me) {
          if (CUT && sh && a.Cpart != nullptr) {
            float* part = a.Cpart + ((size_t)eg * a.shared_rows + m) * N + n0 + 4 * q;
            *reinterpret_cast<float4*>(part) = make_float4(acc0[mt][0], acc0[mt][1], acc0[mt][2], acc0[mt][3]);
            *reinterpret_cast<float4*>(part + 16) = make_float4(acc1[mt][0], acc1[mt][1], acc1[mt][2], acc1[mt][3]);
            continue;
          }
          bf16_t* crow_out = Cb + (size_t)(rb + m) * ldc + n0 + 4 * q;
          uint2 o;
          if (GATEUP) {
            float v[4];
#pragma unroll
            for (int j = 0; j < 4; ++j) v[j] = __fdividef(acc0[mt][j], 1.0f + __expf(-acc0[mt][j])) * acc1[mt][j];
            o.x = pack_bf16x2(v[0], v[1]);
            o.y = pack_bf16x2(v[2], v[3]);
            *reinterpret_cast<uint2*>(crow_out) = o;
          } else {
            o.x = pack_bf16x2(acc0[mt][0], acc0[mt][1]);
            o.y = pack_bf16x2(acc0[mt][2], acc0[mt][3]);
            *reinterpret_cast<uint2*>(crow_out) = o;
            o.x = pack_bf16x2(acc1[mt][0], acc1[mt][1]);
            o.y = pack_bf16x2(acc1[mt][2], acc1[mt][3]);
            *reinterpret_cast<uint2*>(crow_out + 16) = o;
          }
        }
      }
    };
    // multiply the stage in `slot`; `then` runs after the operands are in registers and before the
    // MFMAs (the place to reuse the ring slot that was read one step earlier)
    auto consume = [&](int slot, auto&& then) {
      const unsigned char* st = smem + slot * S::STAGE + frag_off;
      u32x4 w0[2], w1[2], xf[MT][2];
#pragma unroll
      for (int j = 0; j < 2; ++j) {
        const int c = ((4 * j + q) ^ swz) << 4;
        w0[j] = *reinterpret_cast<const u32x4*>(st + c);
        w1[j] = *reinterpret_cast<const u32x4*>(st + 2048 + c);
#pragma unroll
        for (int mt = 0; mt < MT; ++mt) xf[mt][j] = *reinterpret_cast<const u32x4*>(st + S::WBYTES + mt * 2048 + c);
      }
      // the empty asm makes the compiler wait for the LDS reads here: after it the slot may be overwritten
#pragma unroll
      for (int j = 0; j < 2; ++j) {
        asm volatile("" : "+v"(w0[j]));
        asm volatile("" : "+v"(w1[j]));
#pragma unroll
        for (int mt = 0; mt < MT; ++mt) asm volatile("" : "+v"(xf[mt][j]));
      }
      then();
#pragma unroll
      for (int j = 0; j < 2; ++j)
#pragma unroll
        for (int mt = 0; mt < MT; ++mt) {
          acc0[mt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(as_bf16x8(w0[j]), as_bf16x8(xf[mt][j]), acc0[mt], 0, 0, 0);
          acc1[mt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(as_bf16x8(w1[j]), as_bf16x8(xf[mt][j]), acc1[mt], 0, 0, 0);
        }
    };

    f32x4 sum0[MT], sum1[MT];   // (TURN: of the parts before)
    for (int part = part0; part < part1; ++part) {
      if (CUT && sh) {
        nk = a.part_steps + (part < a.part_extra ? 1 : 0);
        kofs = (size_t)(part * a.part_steps + min(part, a.part_extra)) * 128;
        rot = start(blockIdx.x, (unsigned)part);
      }
#pragma unroll
      for (int mt = 0; mt < MT; ++mt) {
        acc0[mt] = f32x4{0.f, 0.f, 0.f, 0.f};
        acc1[mt] = f32x4{0.f, 0.f, 0.f, 0.f};
      }
      if (nk > S::D) {
  #pragma unroll
        for (int s = 0; s < S::D; ++s) issue(s, s);
        int slot = 0;
        for (int s = 0; s + S::D < nk; ++s) {
          wait_copies_but<(S::D - 1) * S::NI>();          // step s has landed
          const int free_slot = slot == 0 ? NST - 1 : slot - 1;   // read one step ago (or never used yet)
          consume(slot, [&] { issue(s + S::D, free_slot); });
          slot = slot + 1 == NST ? 0 : slot + 1;
        }
        stream_tail<0, S::D, S::NI>([&](int) {
          consume(slot, [] {});
          slot = slot + 1 == NST ? 0 : slot + 1;
        });
      } else {   // fewer K steps than ring stages: one stage at a time
        for (int s = 0; s < nk; ++s) {
          issue(s, 0);
          wait_copies_but<0>();
          consume(0, [] {});
        }
      }
      if constexpr (TURN) {
#pragma unroll
        for (int mt = 0; mt < MT; ++mt) {
#pragma unroll
          for (int j = 0; j < 4; ++j) {
            acc0[mt][j] = part > part0 ? sum0[mt][j] + acc0[mt][j] : acc0[mt][j];
            acc1[mt][j] = part > part0 ? sum1[mt][j] + acc1[mt][j] : acc1[mt][j];
          }
          sum0[mt] = acc0[mt];
          sum1[mt] = acc1[mt];
        }
      }
    }
    store();
  }
}

constexpr int STREAM_PASS_GROUPS = 8;

template <int MT, bool GATEUP, int NST, bool SHARED, bool TURN = false, bool SORT = false>
static int launch_stream_lds_t(const GemmArgs& a, hipStream_t st) {
  using S = StreamLdsShape<MT, NST>;
  static_assert(NST * S::STAGE <= 64 * 1024, "dynamic LDS without an opt-in attribute");
  auto kern = expert_stream_lds_kernel<MT, GATEUP, NST, SHARED, TURN, SORT>;
  const int nexp = (a.offsets ? a.hi - a.lo : SHARED ? 0 : 1) + (SHARED ? a.n_shared : 0);
  const int per = GATEUP ? 16 : 32;
  const int gx = (a.N + per - 1) / per;
  if (gx <= 0 || nexp <= 0) return 0;
  // workgroups per (expert, column block): enough that an expert holding every row of the batch runs at most
  // about two passes per workgroup, at most STREAM_PASS_GROUPS (from layer-wide sizes only; a row's result does
  // not depend on it).  Measured at the Qwen shape: 8 cost nothing on unbiased batches (T = 16 ... 384) and
  // take a batch whose hot expert holds nearly every token from 172 + 96 us to 141 + 73 us at T = 128 and
  // from 250 + 159 to 180 + 98 us at T = 384; 16 and 32 begin to cost the unbiased batches 5 - 20 %.
  const int passes_max = (a.rows_total + 16 * MT - 1) / (16 * MT);
  const int gz = std::max(1, std::min(STREAM_PASS_GROUPS, passes_max / 2));
  hipLaunchKernelGGL(kern, dim3(gx, nexp + (SORT ? 1 : 0), gz), dim3(64), NST * S::STAGE, st, a);
  return hipGetLastError() == hipSuccess ? 0 : -4;
}

// One tile of 16 rows covers an expert of a few rows; an expert with more takes further passes over its
// weights.  Ring depths from 2 to 8 stages measured the same within noise; 4 leaves room for five to six
// workgroups per CU.  Larger experts go to the wide kernels: from a mean of 6 rows on, where both read the
// weights at the same rate when the batch is even (8.5 rows: 116 + 62 here, 118 + 60 us there) and a hot
// expert of 127 rows, eight passes here and two there, makes 137 + 70 of it here and 122 + 65 us there.
// One weight set (the shared expert) stays here, with two tiles per pass beyond 16 rows (gate/up + down at 32 rows of
// H 2048, Is 5632 12 + 24 us, with one tile 20 + 42), and so do short contractions, with two beyond a mean of 10.
template <bool GATEUP>
static int launch_stream_lds_any(const GemmArgs& a, hipStream_t st) {
  if (a.N % 32 != 0 || a.Kdim % 64 != 0) return -2;
  if (a.offsets != nullptr && !stream_narrow(a.mean_rows, a.Kdim))
    return a.sort_ids != nullptr ? -2 : GATEUP ? launch_stream_wide_gateup(a, st) : launch_stream_wide_down(a, st);
  const bool two = a.offsets != nullptr ? a.mean_rows > 10 : (a.n_shared > 0 ? a.shared_rows : a.rows_fixed) > 16;
  if constexpr (GATEUP) {
    if (a.sort_ids != nullptr) {
      if (a.offsets == nullptr || a.ids != nullptr || a.n_pairs > SORT_HERE_MAX) return -2;
      if (a.n_shared > 0) return two ? -2 : launch_stream_lds_t<1, true, 4, true, false, true>(a, st);   // (it rides up to a mean of 6 rows)
      return two ? launch_stream_lds_t<2, true, 4, false, false, true>(a, st) : launch_stream_lds_t<1, true, 4, false, false, true>(a, st);
    }
  }
  if constexpr (!GATEUP) {
    if (a.n_shared > 0 && a.n_shared != a.shared_parts)
      return two ? launch_stream_lds_t<2, GATEUP, 4, true, true>(a, st) : launch_stream_lds_t<1, GATEUP, 4, true, true>(a, st);
  }
  if (a.n_shared > 0) return two ? launch_stream_lds_t<2, GATEUP, 4, true>(a, st) : launch_stream_lds_t<1, GATEUP, 4, true>(a, st);
  return two ? launch_stream_lds_t<2, GATEUP, 4, false>(a, st) : launch_stream_lds_t<1, GATEUP, 4, false>(a, st);
}
int launch_stream_lds_gateup(const GemmArgs& a, hipStream_t st) { return launch_stream_lds_any<true>(a, st); }
int launch_stream_lds_down(const GemmArgs& a, hipStream_t st) { return launch_stream_lds_any<false>(a, st); }

}  // namespace moe
