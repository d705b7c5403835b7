// Grouped bf16 GEMM on MFMA for expert blocks with many rows per expert (prefill-sized batches).
// FaaSMoE Sec. 3: an expert block holds several experts and computes on the tokens handed to it;
// Sec. 4.1: the tokens of one block arrive as one batch.  Here a block is an expert range
// [lo,hi) and its batch is a contiguous row range, cut per expert by expert_offsets.
//
// Two instantiations of one kernel:
//   gate/up : h[r, n]  = silu(<A[r,:], Wg[e][n,:]>) * <A[r,:], Wu[e][n,:]>      (A = Xp, Kdim = H)
//   down    : Yp[r, n] = <A[r,:], Wd[e][n,:]>                                   (A = h,  Kdim = I)
// Both operands are K-contiguous, so token rows and weight rows are staged the same way.
//
// Work decomposition.  A tile is BM token rows of ONE expert by BN weight rows (gate/up: BN/2 gate
// rows and the matching BN/2 up rows, so the SwiGLU product is formed in registers).  The number
// of tiles depends on expert_offsets, which only the device knows: the kernel is persistent, every
// wave first forms the per-expert tile prefix in registers and then walks tile indices with a
// fixed stride, so there is no host synchronisation and no atomic.  Workgroup b runs on XCD
// b mod 8; the index walk hands each XCD runs of consecutive tiles that share weight and token
// panels, so they meet in that XCD's L2.
//
// Inside a tile: 4 waves (8 for 256x256, below), K steps of 64 through a ring of NS LDS stages.  Both panels are copied
// from global memory straight into LDS (global_load_lds, 16 bytes per lane, no registers in
// between).  Eight lanes fetch one row's 128 bytes, so every request is a whole cache line: with
// 64-byte requests the L2-to-LDS path delivered 27 B/clk per CU, with 128-byte requests 47 B/clk
// (measured), and these kernels live on that path.  NS-1 stages are in flight while one is
// multiplied.  The copies are asynchronous: a wave waits with s_waitcnt vmcnt(n) until only the
// copies of later stages are outstanding, then one workgroup barrier per K step publishes the
// stage.  A stage is multiplied in four 16-wide K slices; operand fragments are double-buffered in
// registers and every LDS read is issued one slice ahead of its use, between the MFMAs of the
// slice before.  A row's eight 16-byte chunks are stored at slot = chunk xor row%8 so the MFMA
// operand reads (32 rows, same chunk) are bank-conflict free.  MFMA 32x32x16 bf16 with the WEIGHT rows as the
// first operand and the TOKEN rows as the second: a lane then owns 4 consecutive output columns
// of one token row per accumulator quad, which makes the bf16 stores 8 bytes wide.
// Single-tile experts: when all rows of an expert fit one tile nobody else reads its weight panel, and
// the launch is a stream of weights from HBM.  Such tiles request their weights with the read-once hint
// and start their walk over K at a step that depends on the expert and the column tile (it wraps around;
// see the weight-streaming kernels for why a common start crowds the memory channels).  The two belong
// together: with the hint the token panel, which the column tiles of an expert now visit at different
// steps, stays in L2.  60 experts of 137 rows, H 2048, I 1408 (692 MB of gate/up weights): 174-195 us
// without either, 166-177 with the rotation alone, 180 with the hint alone, 153-158 with both (down 88-96
// -> 80-84); 52 rows: 152-174 -> 138.  Experts of several tiles share weight panels through L2, which the
// hint throws away (60 experts of 273 rows: 256 -> 293 us): those keep the plain requests.  The start
// depends on nothing but the expert, the column and the tile shape of the layer, so results do not depend on the block cut.
// Waves: one per SIMD with up to 512 registers, except 256x256: two per SIMD (2x4 waves of 128x64).  These read 1.5 times as
// much from LDS (192 of the 256 KB a stage's 2048 MFMA clocks allow for), but tile border and epilogue, which one wave per SIMD
// walks through alone, take half the time: K loops are 90 % of a workgroup's time instead of 83 %.  Gate/up, 4 -> 8 waves:
// 16 384 rows of the shared expert 643 -> 607 us (1.25 PFLOP/s), 60 experts of 1092 rows 788 -> 727, of 300 344 -> 305, of 200
// 212 -> 191; the down projection 297 -> 295, 422 -> 412, 172 -> 166, 104 -> 100.  Smaller shapes gain nothing (128x256 as
// 2x4, 1x8 or 4x2 waves: equal within 2 %, 192x256 slower for the down projection: 87 -> 103 us at 4096 rows): their LDS reads
// grow past the MFMA time, and where experts stream weights the waves wait for memory.
// The 32-row blocks of a tile are dealt to the WAVES_M rows of waves in turn, so that a tile of few rows is halved between
// them: an expert's last tile of 70 of 256 rows is two blocks per wave instead of three and none.  With four waves side by side
// a copy of token rows belongs to one row of waves, and blocks of padding are not copied either.  60 experts of 1092 rows, gate/up
// + down in us, both: 722 + 405 -> 702 + 397.  What is not copied makes no difference by itself: layers in us, all blocks copied ->
// blocks with rows, 32 experts of 1125 rows of H 2560 1036 -> 1019, 60 of 300 of H 2048 519 -> 524, 64 of 234 of H 1536 256 -> 258, of
// 52 to 137 rows equal within 0.7 %.
// Rows past the end of an expert are clamped on load (they recompute the expert's last row) and
// masked on store, which keeps the K loop free of branches.
#include <math.h>
#include <algorithm>
#include <atomic>
#include <type_traits>
#include "common.h"

namespace moe {

template <int BM, int BN, int WAVES_M, int WAVES_N, bool GATEUP, int NS>
struct TileShape {
  static constexpr int BK = 64;
  static constexpr int ROWB = BK * 2;             // bytes per staged row (8 chunks of 16 bytes)
  static constexpr int WTM = BM / WAVES_M;        // token rows per wave
  static constexpr int WTN = BN / WAVES_N;        // weight rows per wave
  static constexpr int TB = WTM / 32;             // 32-row token blocks per wave
  static constexpr int NB = WTN / 32;             // 32-row weight blocks per wave
  // Gate/up with one weight block per wave: its 32 rows are 8 gate rows, the matching 8 up rows, and both again
  // (16 output columns per wave), so a lane still holds gate and up of a column (elements i and i + 4).
  static constexpr bool MIXED = GATEUP && NB == 1;
  static constexpr int NBH = GATEUP && !MIXED ? NB / 2 : NB;
  static constexpr int STAGE = (BM + BN) * ROWB;  // bytes per LDS stage
  static constexpr int NW = WAVES_M * WAVES_N;      // waves per workgroup
  static constexpr int NL = (BM + BN) / (8 * NW);  // 1 KB (8-row) copies per wave and stage
  static constexpr int NLA = BM / (8 * NW);        // the first NLA of them are token rows
  static constexpr int NF = TB + NB;              // operand fragments per wave and 16-wide K slice
  static constexpr int NM = TB * NB;              // MFMAs per wave and 16-wide K slice
  static constexpr int DIST = NS - 1;             // stages in flight while one is being multiplied
  static constexpr int NOUT = GATEUP ? BN / 2 : BN;  // output columns per tile
  static constexpr int GM = 4;                    // token tiles per locality group of the tile walk
  // The NL copies of a stage are requested in three places, so that the address unit of the CU
  // (one copy instruction of 1 KB keeps it busy for about 16 clocks) is not asked for a whole stage
  // within one K slice: ISSUE0 of them while the last slice of the stage that frees the buffer is
  // multiplied, ISSUE1 and ISSUE2 during the first two slices of the next K step.
  // (the pipeline counts with the copies its token blocks need)
  // With four waves side by side copy i < NLA of a wave is part of the i-th token block of the wave's own row of waves: blocks of
  // padding need not be copied either.
  static constexpr bool TRIM = WAVES_N == 4;
  static constexpr int tokens(int tbc) { return TRIM ? tbc : NLA; }             // token copies of a wave with tbc token blocks
  static constexpr int copies(int tbc) { return tokens(tbc) + NL - NLA; }
  static constexpr int copy(int tbc, int q) { return q < tokens(tbc) ? q : q - tokens(tbc) + NLA; }   // its q-th one
  static_assert(!TRIM || NLA == WTM / 32, "a copy of the token rows is a block of the wave's row");
  static_assert(NW == 4 || NW == 8, "one or two waves per SIMD");
  static_assert(WTM % 32 == 0 && WTN % 32 == 0, "wave tile is made of 32x32 blocks");
  static_assert(!GATEUP || NB == 1 || NB % 2 == 0, "gate and up blocks come in pairs");
  static_assert(BM % (8 * NW) == 0 && BN % (16 * NW) == 0, "copies of 8 rows are dealt to the waves");
  static_assert((NS - 1) * NL < 64, "the wait counter holds 6 bits");
};

constexpr int TILE_EMAX = 256;

// Order in which the operand fragments of a K slice are read: by the MFMA that needs them first.
// MFMA j of a slice multiplies weight block j % NB with token block j / NB, so weight block 0 and
// token block 0 come first, then the other weight blocks, then the token blocks.  Returns the
// fragment number in the numbering "token blocks 0..TB-1, then weight blocks".
__host__ __device__ constexpr int fragment_read_order(int slot, int tb, int nb) {
  return slot == 0 ? tb : (slot == 1 ? 0 : (slot <= nb ? tb + slot - 1 : slot - nb));
}

// KSPLIT > 1: K is cut into that many parts.  Each is a work item whose fp32 sums go to a.Cpart; INTURN: a tile walks all of
// K, sets its sums aside at the end of a part and adds them in the order of the kernel that adds the parts otherwise:
// the same bits without room for the parts, in the time of the uncut tile.
template <int BM, int BN, int WAVES_M, int WAVES_N, bool GATEUP, int NS, int OCC, int KSPLIT, bool SINGLE, bool INTURN>
__global__ __launch_bounds__(64 * WAVES_M * WAVES_N, OCC * WAVES_M * WAVES_N / 4) void expert_tile_kernel(GemmArgs a) {
  using S = TileShape<BM, BN, WAVES_M, WAVES_N, GATEUP, NS>;
  extern __shared__ __align__(16) unsigned char smem[];
  // Experts come in two classes.  One with at least HEAVY_MIN token tiles reuses every weight panel
  // that often out of L2 and is bound by the matrix pipes; one with fewer streams its weights from
  // HBM for little arithmetic and is bound by memory.  Walking the experts in id order would run
  // long stretches of one kind (all CUs waiting for HBM, then HBM idle); instead the token tiles
  // of each class are listed separately (experts in order inside a class) and the walk draws
  // locality groups from the two lists in proportion, so both kinds are in flight at any time.
  constexpr int HEAVY_MIN = 3;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave / WAVES_N, wn = wave % WAVES_N;
  // weight sets of this launch: the routed experts of the block, then the shared sets riding along
  const int nrouted = a.offsets ? a.hi - a.lo : (a.n_shared > 0 ? 0 : 1);
  const int nexp = nrouted + a.n_shared;     // at most TILE_EMAX (checked by the caller)

  // Row range and token tiles of four experts per lane: [first[i], last[i]) in the tiles of the expert's class, rows
  // [rb[i], re[i]).  Every wave keeps all of it in registers, where finding the expert of a tile is a handful of compares and
  // ballots: a workgroup has one or two waves per SIMD, so what it waits for at a tile border little else fills.  (As prefixes in LDS
  // and a binary search, with the expert's end re-read from memory: gate/up + down in us
  // 60 experts of H 2048, I 1408 at 33, 51, 273 and 546 rows 131+67, 138+73, 257+135, 421+246; so 128+66, 134+71, 255+133, 415+241.)
  int first[4], last[4], rb[4], re[4], cnt[2] = {0, 0};
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int e = lane * 4 + i;
    rb[i] = re[i] = 0;
    if (e < nexp) {
      const bool sh = e >= nrouted;
      const int eid = sh ? e - nrouted : (a.offsets ? (a.ids ? a.ids[a.lo + e] : a.lo + e) : 0);
      rb[i] = sh ? a.rows_routed + eid * a.shared_rows : (a.offsets ? a.offsets[eid] : 0);
      re[i] = sh ? rb[i] + a.shared_rows : (a.offsets ? a.offsets[eid + 1] : a.rows_fixed);
    }
    last[i] = (max(re[i] - rb[i], 0) + BM - 1) / BM;      // (a count so far)
    cnt[last[i] >= HEAVY_MIN] += last[i];
  }
  int total[2];
#pragma unroll
  for (int c = 0; c < 2; ++c) {
    int incl = cnt[c];
#pragma unroll
    for (int s = 1; s < 64; s <<= 1) {
      const int o = __shfl_up(incl, s, WAVE);
      if (lane >= s) incl += o;
    }
    total[c] = __builtin_amdgcn_readlane(incl, 63);
    cnt[c] = incl - cnt[c];                               // tiles of this class before this lane's experts
  }
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const bool heavy = last[i] >= HEAVY_MIN;
    first[i] = heavy ? cnt[1] : cnt[0];
    last[i] += first[i];
    cnt[0] = heavy ? cnt[0] : last[i];
    cnt[1] = heavy ? last[i] : cnt[1];
  }
  const int total0 = total[0], total1 = total[1];
  const int grp0 = (total0 + S::GM - 1) / S::GM, grp1 = (total1 + S::GM - 1) / S::GM;   // locality groups per class
  const int ngrp = grp0 + grp1;
  const int NT = (a.N + S::NOUT - 1) / S::NOUT;
  const int Kdim = a.Kdim;
  constexpr int ITEMS = INTURN ? 1 : KSPLIT;     // work items of a tile
  const int nk = Kdim / S::BK / ITEMS;           // K steps of one work item (a tile, or a K part of it)
  const int groupTiles = S::GM * NT;
  // With one class the walk ends with its last tile.  (With two, the incomplete last group of each leaves a
  // gap; tiles of a complete index space that do not exist would otherwise push real ones into one more round:
  // 777 tokens on one weight set are 5 tiles of 160 rows by 44 column tiles, 220 for 256 workgroups, and took
  // 73 us as 8 x 44 with gaps.)
  const int Lend = (grp0 == 0 || grp1 == 0 ? (total0 + total1) * NT : ngrp * groupTiles) * ITEMS;
  // Divisions of the walk, prepared once per workgroup so that finding a tile costs multiplications only:
  // light groups among the first g groups of the merged walk = (g * light_ratio) >> 32, with light_ratio =
  // ceil(grp0 * 2^32 / ngrp): monotone in g, rises by at most one per group, and is exactly grp0 at g = ngrp,
  // so every group of either class is drawn exactly once; x / groupTiles and pair / gather_div by a
  // multiply-high with one correction step.
  const unsigned long long light_ratio = ngrp > 0 ? ((((unsigned long long)grp0) << 32) + (unsigned)ngrp - 1ull) / (unsigned)ngrp : 0ull;
  const uint32_t gt_magic = groupTiles > 1 ? (uint32_t)(0x100000000ull / (unsigned)groupTiles) : 0u;   // (2^32 itself does not fit)
  const uint32_t gd = a.gather ? (uint32_t)a.gather_div : 1u;
  const uint32_t gd_magic = gd > 1u ? (uint32_t)(0x100000000ull / gd) : 0u;

  const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) unsigned char*)smem;
  // copy assignment of this lane inside an 8-row block: row lane/8, 16-byte slot lane%8; the slot
  // holds chunk (slot xor row%8) of the row, which spreads the MFMA operand reads (32 rows at the
  // same chunk) over all banks.
  const int crow = lane >> 3;
  const int cchunk = (lane & 7) ^ (lane >> 3);
  // operand reads: row lane%32 of a 32-row block, chunk 2*kk + lane/32 of the row
  const int frag_row = lane & 31;
  const int wfrag_row = S::MIXED ? ((frag_row >> 3) & 1) * (BN / 2) + (frag_row >> 4) * 8 + (frag_row & 7) : frag_row;
  const int frag_half = lane >> 5;
  const int frag_swz = lane & 7;

  // Tile walk.  Workgroup b runs on XCD b % 8.  Each XCD takes runs of `run` consecutive tile
  // indices (tiles that share panels), one per workgroup slot; with fewer tiles than slots the runs
  // shrink so that all eight XCDs still get an equal share.
  const int G = gridDim.x;
  const bool xcd_walk = (G % 8) == 0;
  const int slot = xcd_walk ? (int)(blockIdx.x >> 3) : 0;
  const int run = xcd_walk ? max(1, min(G >> 3, (Lend + 7) >> 3)) : 1;
  if (xcd_walk && slot >= run) return;

    // copy i (of NL) of K step kt into stage buffer st; all NL of them.  once_: the weight rows carry the
    // read-once hint (see "single-tile experts" above)
#define MOE_TILE_ISSUE1(kt, st, i, once_)                                                           \
    copy_to_lds_16(                                                                                 \
        ((i) < S::NLA ? Ag : ((GATEUP && (i) >= S::NLA + (S::NL - S::NLA) / 2) ? Bg1 : Bg0)) + (size_t)(kt) * S::ROWB, \
        coff[i], lds0 + (uint32_t)(st) * S::STAGE + (uint32_t)wave * 1024u + (uint32_t)(i) * (S::NW * 1024u), (once_) && (i) >= S::NLA);

  // State of a tile: the current one (being multiplied, then stored) and, while the current one is
  // stored, the next one, whose first NS stages are already requested: the latency of those copies
  // hides behind the epilogue instead of opening every tile.
  struct TileState { int row0, rowEnd, rowsValid, tbv, n0, ks, cshift, ncols, ldc; bf16_t* cbase; bool once, valid; };
  const unsigned char *Ag = nullptr, *Bg0 = nullptr, *Bg1 = nullptr;
  uint32_t coff[S::NL];   // byte offsets of this lane's 16 bytes for each of the NL copies of a stage (K step 0)
  int krot = 0;           // K step the tile starts at (its walk over K wraps around)
  auto kstep = [&](int kt) -> int { const int k = kt + krot; return k >= nk ? k - nk : k; };
  int it = 0;
  auto next_tile = [&]() -> TileState {
    // The arguments are read again for every tile: kept over the K loops they would not fit the scalar registers, and what is
    // set aside in vector lanes comes back one wait at a time.
    const __attribute__((address_space(4))) GemmArgs* args = (const __attribute__((address_space(4))) GemmArgs*)__builtin_amdgcn_kernarg_segment_ptr();
    asm volatile("" : "+s"(args));
    const auto& a = *args;
    TileState t{};
    int L = 0, mrow = 0, nt = 0, cls = 0, ks = 0;
    for (;; ++it) {
      L = xcd_walk ? ((it * 8 + (int)(blockIdx.x & 7)) * run + slot) : (it * G + (int)blockIdx.x);
      if (L >= Lend) { t.valid = false; return t; }
      int Lt = L;
      ks = 0;
      if constexpr (ITEMS > 1) {   // K parts outermost: the items of an XCD share panels, not only sums
        const int tiles = Lend / ITEMS;
        while (Lt >= tiles) { Lt -= tiles; ++ks; }
      }
      int grp = Lt, rem = 0;
      if (groupTiles > 1) {
        grp = (int)__umulhi((uint32_t)Lt, gt_magic);   // floor(2^32/d) underestimates the quotient by at most one
        rem = Lt - grp * groupTiles;
        if (rem >= groupTiles) { ++grp; rem -= groupTiles; }
      }
      // group grp of the merged walk: light groups are spread evenly between the heavy ones
      const int before = (int)(((unsigned long long)(unsigned)grp * light_ratio) >> 32);          // light groups among the first grp
      cls = (int)(((unsigned long long)(unsigned)(grp + 1) * light_ratio) >> 32) > before ? 0 : 1;
      const int first = (cls == 0 ? before : grp - before) * S::GM;      // first token tile of the group
      const int size = min(S::GM, (cls == 0 ? total0 : total1) - first);    // its token tiles
      if (size == S::GM) {
        nt = rem / S::GM;
        mrow = first + rem % S::GM;
      } else {
        nt = rem / size;
        mrow = first + rem - nt * size;
      }
      if (nt < NT) break;
    }
    ++it;
    t.valid = true;
    t.ks = ks;   // K part of this work item

    // the expert of this token tile: exactly one lane and i (the same in every lane: scalar registers)
    int at = 0, vf = 0, vb = 0, ve = 0;
    unsigned long long found = 0ull;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const bool own = (last[i] - first[i] >= HEAVY_MIN) == (cls == 1) && first[i] <= mrow && mrow < last[i];
      found |= __ballot(own);
      at = own ? i : at;
      vf = own ? first[i] : vf;
      vb = own ? rb[i] : vb;
      ve = own ? re[i] : ve;
    }
    const int owner = __builtin_ctzll(found);
    const int e = owner * 4 + __builtin_amdgcn_readlane(at, owner);
    const bool sh = e >= nrouted;
    const int eg = sh ? e - nrouted : a.ids ? a.ids[a.lo + e] : a.offsets ? a.lo + e : 0;   // expert id, or the number of the shared set
    const int rb_e = __builtin_amdgcn_readlane(vb, owner);
    t.row0 = rb_e + (mrow - __builtin_amdgcn_readlane(vf, owner)) * BM;
    t.rowEnd = __builtin_amdgcn_readlane(ve, owner);
    t.rowsValid = min(BM, t.rowEnd - t.row0);
    // token blocks of this wave that hold rows of the expert (at least one, so that the copies and
    // operand reads keep their places between MFMAs)
    t.tbv = min(S::TB, max(1, (((t.rowsValid + 31) >> 5) - wm + WAVES_M - 1) / WAVES_M));
    t.n0 = nt * S::NOUT;
    t.once = SINGLE && t.rowEnd - rb_e <= BM;
    // where this tile's rows go: a shared set may have an output tensor of its own
    const bool own_c = sh && a.Cs != nullptr;
    const bool of_one = GATEUP && own_c && a.shared_cols != 0;    // the sets are columns of one hidden layer
    t.cbase = own_c ? a.Cs + (of_one ? (size_t)eg * a.N : (size_t)0) : a.C;
    t.cshift = of_one ? rb_e : own_c ? a.rows_routed : 0;
    t.ldc = of_one ? a.shared_cols : a.N;
    // (a column tile of a narrower last set may lie past its columns: it repeats the last one and stores nothing)
    t.ncols = of_one ? min(a.N, a.shared_cols - eg * a.N) : a.N;

    const size_t kbeg = (size_t)t.ks * nk * S::BK;
    // token rows: with a gather list they are addressed from the start of A, through the list; a
    // shared set with token rows of its own reads them in order
    const bool own_a = sh && a.As != nullptr;
    const bool gathered = a.gather != nullptr && !own_a;
    Ag = reinterpret_cast<const unsigned char*>(
        own_a ? a.As + (size_t)(t.row0 - rb_e) * Kdim + kbeg : a.A + (gathered ? (size_t)0 : (size_t)t.row0 * Kdim) + kbeg);
    const uint32_t ldb = sh ? (uint32_t)a.ldb_shared : (uint32_t)Kdim;   // elements between consecutive weight rows
    Bg0 = reinterpret_cast<const unsigned char*>((sh ? a.Bs0 + (size_t)eg * a.shared_b_step : a.B0 + (size_t)eg * a.N * Kdim) + kbeg);
    Bg1 = GATEUP ? reinterpret_cast<const unsigned char*>((sh ? a.Bs1 + (size_t)eg * a.shared_b_step : a.B1 + (size_t)eg * a.N * Kdim) + kbeg)
                 : nullptr;
#pragma unroll
    for (int i = 0; i < S::NL; ++i) {
      const int row = (i * S::NW + wave) * 8 + crow;        // row inside the stage: tokens first, then weights
      int grow;
      uint32_t ld = (uint32_t)Kdim;
      if (i < S::NLA) {
        grow = min(row, t.rowsValid - 1);
        if (gathered) {
          const uint32_t pair = (uint32_t)a.gather[t.row0 + grow];
          uint32_t tok = pair;
          if (gd > 1u) {
            tok = __umulhi(pair, gd_magic);
            if (pair - tok * gd >= gd) ++tok;
          }
          grow = (int)tok;
        }
      } else {
        int r = row - BM;
        if (GATEUP && i >= S::NLA + (S::NL - S::NLA) / 2) r -= BN / 2;   // second half: the up branch
        grow = min(t.n0 + r, t.ncols - 1);
        ld = ldb;
      }
      coff[i] = (uint32_t)grow * ld * 2u + (uint32_t)cchunk * 16u;
    }
    // all NS stages of the tile are requested up front
    auto request = [&](auto once_) {
#pragma unroll
      for (int s = 0; s < NS; ++s) {
        const int k = decltype(once_)::value ? kstep(min(s, nk - 1)) : min(s, nk - 1);
#pragma unroll
        for (int i = 0; i < S::NL; ++i)
          if (!S::TRIM || i >= S::NLA || i < t.tbv) MOE_TILE_ISSUE1(k, s, i, decltype(once_)::value);
      }
    };
    if (SINGLE && t.once) {
      krot = (int)((unsigned)(eg * 5 + (t.n0 >> a.rot_shift) * 3) % (unsigned)nk);
      request(std::true_type{});
    } else {
      request(std::false_type{});
    }
    return t;
  };

  // Clock record of this workgroup (a measurement aid).  The clocks are read whether or not a record was asked
  // for (two scalar reads per tile): a branch between a K loop's last MFMAs and the epilogue's first read of the
  // accumulators would sit exactly where the compiler has to pad that pair with wait states, and it does not
  // look across such a branch (build.py checks the emitted code for this).  Only the final store is conditional.
  const bool clocked = a.clocks != nullptr && (int)blockIdx.x < a.clock_groups;
  long long clk_kloops = 0, clk_tiles = 0;
  const long long clk_begin = clock64(), wall_begin = wall_clock64();

  f32x16 sum[INTURN ? S::NB : 1][INTURN ? S::TB : 1];   // of the K parts before (INTURN)
  TileState cur = next_tile();
  while (cur.valid) {
    const int row0 = cur.row0, rowEnd = cur.rowEnd, n0 = cur.n0, ks = cur.ks;
    bf16_t* const cbase = cur.cbase;
    const int cshift = cur.cshift, ldc = cur.ldc, ncols = cur.ncols;
    f32x16 acc[S::NB][S::TB];
#pragma unroll
    for (int nb = 0; nb < S::NB; ++nb)
#pragma unroll
      for (int tb = 0; tb < S::TB; ++tb)
#pragma unroll
        for (int i = 0; i < 16; ++i) acc[nb][tb][i] = 0.0f;

    // fragment f of the 16-wide K slice kk_ of a stage, LDS -> registers: f < TBc is the token block
    // f, otherwise the weight block f - TBc.  TBc <= TB is the number of 32-row token blocks of this
    // wave that hold rows of the expert: blocks of pure padding are neither read nor multiplied.
#define MOE_TILE_READ1(fa_, fb_, stage_, kk_, f_)                                                   \
    {                                                                                               \
      const unsigned char* As_ = smem + (stage_) * S::STAGE;                                         \
      const int cr_ = (((kk_) * 2 + frag_half) ^ frag_swz) << 4;                                     \
      if ((f_) < TBc) {                                                                             \
        fa_[(f_) < TBc ? (f_) : 0] = as_bf16x8(*reinterpret_cast<const u32x4*>(                    \
            As_ + (((f_) * WAVES_M + wm) * 32 + frag_row) * S::ROWB + cr_));                         \
      } else {                                                                                      \
        const int nb_ = (f_) < TBc ? 0 : (f_) - TBc;                                                \
        const int brow_ = S::MIXED ? wn * 16 : GATEUP ? ((nb_ < S::NBH ? 0 : BN / 2) + wn * (S::WTN / 2) + (nb_ % S::NBH) * 32) \
                                 : (wn * S::WTN + nb_ * 32);                                         \
        fb_[nb_] = as_bf16x8(*reinterpret_cast<const u32x4*>(                                        \
            As_ + BM * S::ROWB + (brow_ + wfrag_row) * S::ROWB + cr_));                              \
      }                                                                                             \
    }
#define MOE_TILE_READ(fa_, fb_, stage_, kk_)                                                        \
    { _Pragma("unroll") for (int f = 0; f < NFc; ++f) MOE_TILE_READ1(fa_, fb_, stage_, kk_, f); }
#define MOE_TILE_MFMA1(fa_, fb_, j_)                                                                \
    acc[(j_) % S::NB][(j_) / S::NB] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(                       \
        fb_[(j_) % S::NB], fa_[(j_) / S::NB], acc[(j_) % S::NB][(j_) / S::NB], 0, 0, 0);
#define MOE_TILE_MMA(fa_, fb_)                                                                      \
    { _Pragma("unroll") for (int j = 0; j < NMc; ++j) MOE_TILE_MFMA1(fa_, fb_, j); }
    // One K slice: multiply the fragments in set X and, spread between the MFMAs, read the
    // fragments of slice kk_ of stage_ into set Y.  The scheduling fences pin that interleaving, so
    // no LDS read is issued in front of an idle matrix pipe.
#define MOE_TILE_SLICE(faX, fbX, faY, fbY, stage_, kk_)                                             \
    { _Pragma("unroll") for (int j = 0; j < NMc; ++j) {                                             \
        MOE_TILE_MFMA1(faX, fbX, j);                                                                \
        _Pragma("unroll") for (int f = 0; f < NFc; ++f)                                             \
          if (f * NMc / NFc == j) MOE_TILE_READ1(faY, fbY, stage_, kk_, fragment_read_order(f, TBc, S::NB)); \
        __builtin_amdgcn_sched_barrier(0x6);                                                        \
    } }
    // The same with copies I0 .. I1-1 of K step kt_issue_ (into buffer st_issue_) requested in between.
#define MOE_TILE_SLICE_ISSUE(faX, fbX, faY, fbY, stage_, kk_, kt_issue_, st_issue_, I0, I1)         \
    { _Pragma("unroll") for (int j = 0; j < NMc; ++j) {                                             \
        MOE_TILE_MFMA1(faX, fbX, j);                                                                \
        _Pragma("unroll") for (int q = 0; q < ((I1) - (I0)) + NFc; ++q)                             \
          if (q * NMc / (((I1) - (I0)) + NFc) == j) {                                               \
            constexpr int NE_ = S::NB + 1 < NFc ? S::NB + 1 : NFc;   /* reads needed early: before the copies */ \
            constexpr int NC_ = (I1) - (I0);                                                        \
            if (q < NE_) MOE_TILE_READ1(faY, fbY, stage_, kk_, fragment_read_order(q < NE_ ? q : 0, TBc, S::NB)) \
            else if (q < NE_ + NC_) { MOE_TILE_ISSUE1(kt_issue_, st_issue_, S::copy(TBc, (q >= NE_ && q < NE_ + NC_) ? (I0) + q - NE_ : 0), ONCE); } \
            else MOE_TILE_READ1(faY, fbY, stage_, kk_, fragment_read_order(q >= NE_ + NC_ ? q - NC_ : 0, TBc, S::NB)) \
          }                                                                                         \
        __builtin_amdgcn_sched_barrier(0x6);                                                        \
    } }
    // Last slice of a stage: multiply set B; between the MFMAs first request the first copies of the
    // stage that reuses the buffer just freed, then read slice 0 of the next stage into set A.
#define MOE_TILE_SLICE_LAST(next_stage_, kt_issue_, st_issue_)                                      \
    { _Pragma("unroll") for (int j = 0; j < NMc; ++j) {                                             \
        MOE_TILE_MFMA1(faB, fbB, j);                                                                \
        _Pragma("unroll") for (int q = 0; q < ISSUE0 + NFc; ++q)                                    \
          if (q * NMc / (ISSUE0 + NFc) == j) {                                                      \
            constexpr int NE_ = S::NB + 1 < NFc ? S::NB + 1 : NFc;                                  \
            if (q < NE_) MOE_TILE_READ1(faA, fbA, next_stage_, 0, fragment_read_order(q < NE_ ? q : 0, TBc, S::NB)) \
            else if (q < NE_ + ISSUE0) { MOE_TILE_ISSUE1(kt_issue_, st_issue_, S::copy(TBc, (q >= NE_ && q < NE_ + ISSUE0) ? q - NE_ : 0), ONCE); } \
            else MOE_TILE_READ1(faA, fbA, next_stage_, 0, fragment_read_order(q >= NE_ + ISSUE0 ? q - ISSUE0 : 0, TBc, S::NB)) \
          }                                                                                         \
        __builtin_amdgcn_sched_barrier(0x6);                                                        \
    } }

    // Pipeline.  All NS stages have been requested (next_tile); while stage kt is multiplied, stages
    // kt+1 .. kt+NS-1 are in flight.  Fragment sets A and B alternate over the four slices of a
    // stage; slice 0 of the NEXT stage is read (after the barrier that publishes it) while the last
    // slice is multiplied.  That barrier also tells every wave that stage kt has been read
    // completely, so its buffer can take the copy of stage kt+NS.
    // (Past the end of K the requests repeat the last K step into a buffer nobody reads again:
    // every iteration then issues the same number of copies and the wait counts stay constant.)
    auto pipeline = [&](auto tbc_, auto once_) {
      constexpr int TBc = decltype(tbc_)::value;
      constexpr bool ONCE = decltype(once_)::value;
      constexpr int NMc = TBc * S::NB;   // MFMAs per 16-wide K slice
      constexpr int NFc = TBc + S::NB;   // operand fragments per slice
      constexpr int NLc = S::copies(TBc);   // copies per stage
      constexpr int ISSUE0 = NLc - 2 * (NLc / 3), ISSUE1 = NLc / 3;
      wait_copies_but<S::DIST * NLc>();   // stage 0 (requested before the previous tile was stored) has landed
      workgroup_barrier();
      bf16x8 faA[S::TB], fbA[S::NB], faB[S::TB], fbB[S::NB];
      MOE_TILE_READ(faA, fbA, 0, 0);
      int st = 0;                                  // buffer of the stage being multiplied: kt % NS
      int part_end = nk / KSPLIT;                  // (INTURN) K step at which the part ends
      for (int kt = 0; kt + 1 < nk; ++kt) {
        const int st1 = st + 1 == NS ? 0 : st + 1;
        // the rest of the copies of K step kt-1+NS, whose first part went out during the last slice
        // of K step kt-1 (at kt = 0 this repeats copies of the prologue: same bytes, same place)
        const int ktd = ONCE ? kstep(min(kt - 1 + NS, nk - 1)) : min(kt - 1 + NS, nk - 1);
        const int std_ = st == 0 ? NS - 1 : st - 1;
        MOE_TILE_SLICE_ISSUE(faA, fbA, faB, fbB, st, 1, ktd, std_, ISSUE0, ISSUE0 + ISSUE1);
        MOE_TILE_SLICE_ISSUE(faB, fbB, faA, fbA, st, 2, ktd, std_, ISSUE0 + ISSUE1, NLc);
        MOE_TILE_SLICE(faA, fbA, faB, fbB, st, 3);
        // this wave has finished reading stage kt once the last-slice fragments are in registers
        // (the empty asm makes the compiler wait for them; the fence keeps that wait behind the MFMAs)
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int tb = 0; tb < TBc; ++tb) asm volatile("" : "+v"(faB[tb]));
#pragma unroll
        for (int nb = 0; nb < S::NB; ++nb) asm volatile("" : "+v"(fbB[nb]));
        wait_copies_but<(S::DIST - 1) * NLc>();
        workgroup_barrier();  // stage kt+1 is complete for everyone; stage kt is free for everyone
        MOE_TILE_SLICE_LAST(st1, ONCE ? kstep(min(kt + NS, nk - 1)) : min(kt + NS, nk - 1), st);
        if constexpr (INTURN) {
          if (kt + 1 == part_end) {   // (the wait states between the slice's last MFMAs and their results: the branch hides the pair)
            asm volatile("s_nop 15\n\ts_nop 15" ::: "memory");
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int nb = 0; nb < S::NB; ++nb)
#pragma unroll
              for (int tb = 0; tb < S::TB; ++tb)
#pragma unroll
                for (int i = 0; i < 16; ++i) {
                  sum[nb][tb][i] = part_end == nk / KSPLIT ? acc[nb][tb][i] : sum[nb][tb][i] + acc[nb][tb][i];
                  acc[nb][tb][i] = 0.0f;
                }
            part_end += nk / KSPLIT;
          }
        }
        st = st1;
      }
      MOE_TILE_SLICE(faA, fbA, faB, fbB, st, 1);
      MOE_TILE_SLICE(faB, fbB, faA, fbA, st, 2);
      MOE_TILE_SLICE(faA, fbA, faB, fbB, st, 3);
      MOE_TILE_MMA(faB, fbB);
      wait_lds_reads();
      wait_copies_but<0>();  // the repeated last-step copies of the final iterations: none may outlive the tile
      workgroup_barrier();   // the next tile's first copies overwrite stages other waves may still read
    };
    const int tbv = cur.tbv;
    const long long clk_k0 = clock64();
    auto run_pipeline = [&](auto once_) {
      switch (tbv) {
        case 1: pipeline(std::integral_constant<int, 1>{}, once_); break;
        case 2: if constexpr (S::TB >= 2) pipeline(std::integral_constant<int, 2>{}, once_); break;
        case 3: if constexpr (S::TB >= 3) pipeline(std::integral_constant<int, 3>{}, once_); break;
        case 4: if constexpr (S::TB >= 4) pipeline(std::integral_constant<int, 4>{}, once_); break;
        default: if constexpr (S::TB >= 5) pipeline(std::integral_constant<int, 5>{}, once_); break;
      }
    };
    if (SINGLE && cur.once) run_pipeline(std::true_type{}); else run_pipeline(std::false_type{});
    static_assert(S::TB <= 5, "token blocks per wave");
    clk_kloops += clock64() - clk_k0;
    ++clk_tiles;
#undef MOE_TILE_READ1
#undef MOE_TILE_MFMA1
#undef MOE_TILE_SLICE
#undef MOE_TILE_SLICE_LAST
#undef MOE_TILE_SLICE_ISSUE
#undef MOE_TILE_READ
#undef MOE_TILE_MMA

    // the stage buffers are free (final barrier of the pipeline): request the next tile's first
    // stages now, their way from L2 overlaps the stores below
    const TileState nxt = next_tile();

    if constexpr (INTURN) {   // the last part
#pragma unroll
      for (int nb = 0; nb < S::NB; ++nb)
#pragma unroll
        for (int tb = 0; tb < S::TB; ++tb)
#pragma unroll
          for (int i = 0; i < 16; ++i) acc[nb][tb][i] = sum[nb][tb][i] + acc[nb][tb][i];
    }

    // epilogue: accumulator element i of block (nb, tb) is output column
    // 8*(i/4) + 4*(lane/32) + i%4 of the block, token row lane%32: lanes l and l+32 hold the two
    // halves of every 8-column group of a row.  In the down projection the two lanes trade one
    // group each (lane l gives its half of group q+1 and takes the partner's half of group q), so
    // each then owns 8 consecutive columns and stores 16 bytes: half as many store instructions,
    // and a row receives whole 32-byte pieces.  Stores count in the same counter as the copy ring,
    // so the first K steps of the next tile wait for them (without any stores the routed down
    // projection at T=4096 takes 114 instead of 144 us); the wider stores bring it to 134 us.  The
    // gate/up kernels, whose tiles store half as much behind the SwiGLU arithmetic, keep 8-byte
    // stores (16-byte ones: equal for the routed experts, 2 % slower for the shared one).
    auto out_value = [&](int nb, int tb, int i) -> float {
      if (GATEUP) {
        const float g = acc[nb][tb][i];
        const float u = S::MIXED ? acc[nb][tb][i + 4 < 16 ? i + 4 : i] : acc[S::MIXED ? nb : nb + S::NBH][tb][i];
        return __fdividef(g, 1.0f + __expf(-g)) * u;
      }
      return acc[nb][tb][i];
    };
#pragma unroll
    for (int tb = 0; tb < S::TB; ++tb) {
      const int m = row0 + (tb * WAVES_M + wm) * 32 + frag_row;
      if (m < rowEnd) {
        bf16_t* crow_out = cbase + (size_t)(m - cshift) * ldc;
#pragma unroll
        for (int nb = 0; nb < S::NBH; ++nb) {
          const int nblock = n0 + (GATEUP ? wn * (S::WTN / 2) : wn * S::WTN) + nb * 32;   // first column of the 32-column block
          if (nblock < ncols) {   // N is a multiple of 64, nblock of 32 (of 16, and 16 columns, for MIXED): inside or outside as a whole
            if (ITEMS > 1) {   // fp32 partial sum of K part ks; summed in order by the reduce kernel
#pragma unroll
              for (int q = 0; q < 4; ++q) {
                const int n = nblock + 4 * frag_half + 8 * q;
                float* part = a.Cpart + ((size_t)ks * a.rows_total + m) * a.N + n;
                *reinterpret_cast<float4*>(part) = make_float4(out_value(nb, tb, 4 * q), out_value(nb, tb, 4 * q + 1),
                                                               out_value(nb, tb, 4 * q + 2), out_value(nb, tb, 4 * q + 3));
              }
            } else if (GATEUP) {
#pragma unroll
              for (int q = 0; q < 4; q += S::MIXED ? 2 : 1) {
                uint2 o;
                o.x = pack_bf16x2(out_value(nb, tb, 4 * q), out_value(nb, tb, 4 * q + 1));
                o.y = pack_bf16x2(out_value(nb, tb, 4 * q + 2), out_value(nb, tb, 4 * q + 3));
                *reinterpret_cast<uint2*>(crow_out + nblock + 4 * frag_half + (S::MIXED ? 4 : 8) * q) = o;
              }
            } else {
#pragma unroll
              for (int q = 0; q < 4; q += 2) {
                uint32_t ox = pack_bf16x2(out_value(nb, tb, 4 * q), out_value(nb, tb, 4 * q + 1));
                uint32_t oy = pack_bf16x2(out_value(nb, tb, 4 * q + 2), out_value(nb, tb, 4 * q + 3));
                uint32_t oz = pack_bf16x2(out_value(nb, tb, 4 * q + 4), out_value(nb, tb, 4 * q + 5));
                uint32_t ow = pack_bf16x2(out_value(nb, tb, 4 * q + 6), out_value(nb, tb, 4 * q + 7));
                // (x,y) = own half of group q, (z,w) = own half of group q+1.  After the trade lanes 0-31
                // hold group q complete in (x,y,z,w), lanes 32-63 group q+1.
                trade_halves(ox, oz);
                trade_halves(oy, ow);
                *reinterpret_cast<u32x4*>(crow_out + nblock + 8 * (q + frag_half)) = u32x4{ox, oy, oz, ow};
              }
            }
          }
        }
      }
    }
    cur = nxt;
  }
#undef MOE_TILE_ISSUE1
  if (clocked && tid == 0) {
    long long* rec = a.clocks + 4 * (size_t)blockIdx.x;
    rec[0] = clock64() - clk_begin;
    rec[1] = wall_clock64() - wall_begin;
    rec[2] = clk_kloops;
    rec[3] = clk_tiles;
  }
}

static thread_local long long* t_clock_buffer = nullptr;
static thread_local int t_clock_groups = 0;
void set_tile_clock_buffer(long long* clocks, int groups) {
  t_clock_buffer = groups > 0 ? clocks : nullptr;
  t_clock_groups = clocks != nullptr && groups > 0 ? groups : 0;
}

// Compute units of the current device (asked on every launch: nothing is cached across devices or threads).
static int num_cus() {
  int dev = 0, n = 0;
  if (hipGetDevice(&dev) != hipSuccess) return 256;
  if (hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || n <= 0) return 256;
  return n;
}

template <int BM, int BN, int WAVES_M, int WAVES_N, bool GATEUP, int NS, int OCC, int KSPLIT, bool SINGLE, bool INTURN = false>
static int launch_tile_s(const GemmArgs& a, hipStream_t st) {
  using S = TileShape<BM, BN, WAVES_M, WAVES_N, GATEUP, NS>;
  auto kern = expert_tile_kernel<BM, BN, WAVES_M, WAVES_N, GATEUP, NS, OCC, KSPLIT, SINGLE, INTURN>;
  static_assert(std::is_same<decltype(kern), void (*)(GemmArgs)>::value, "next_tile reads the arguments at the start of the kernel's");
  static_assert(KSPLIT == 1 || !SINGLE, "a K part of a tile does not wrap around");
  static_assert(KSPLIT == 1 || !GATEUP, "the SwiGLU product needs complete sums");
  if (a.Kdim % (S::BK * KSPLIT) != 0) return -2;
  if (KSPLIT > 1 && !INTURN && a.Cpart == nullptr) return -3;
  static_assert(OCC * NS * S::STAGE <= 160 * 1024, "LDS of the resident workgroups must fit a CU");
  static std::atomic<uint64_t> lds_raised{0};
  const int lds = NS * S::STAGE;
  if (raise_lds_limit((const void*)kern, lds, lds_raised) != 0) return -4;
  const int nexp = (a.offsets ? a.hi - a.lo : (a.n_shared > 0 ? 0 : 1)) + a.n_shared;
  if (nexp > TILE_EMAX) return -2;
  const int NT = (a.N + S::NOUT - 1) / S::NOUT;
  const long mt_bound = (long)a.rows_total / BM + nexp;
  const long bound = ((mt_bound + S::GM - 1) / S::GM) * S::GM * NT * (INTURN ? 1 : KSPLIT);
  // persistent workgroups: as many as fit on the chip at once (two per CU for the smaller tile)
  const long resident = (long)num_cus() * OCC;
  int grid = (int)(bound < resident ? bound : resident);
  if (grid <= 0) return 0;
  GemmArgs launched = a;
  launched.clocks = t_clock_buffer;
  launched.clock_groups = t_clock_groups;
  hipLaunchKernelGGL(kern, dim3(grid), dim3(64 * S::NW), lds, st, launched);
  return hipGetLastError() == hipSuccess ? 0 : -4;
}

// Batches whose mean expert needs more than four tiles hold (next to) no single-tile expert: they run the
// instance without that path (with it the 256x256 kernels at 16 384 tokens lose 0.6 %, to registers and code
// that no tile uses), and so does one weight set (the shared expert; with one token its gate/up kernel takes
// 2 us more with the path than without).  The rule reads layer-wide sizes only.
template <int BM, int BN, int WAVES_M, int WAVES_N, bool GATEUP, int NS, int OCC>
static int launch_tile_t(const GemmArgs& a, hipStream_t st) {
  if (a.offsets && a.mean_rows <= 4 * BM) return launch_tile_s<BM, BN, WAVES_M, WAVES_N, GATEUP, NS, OCC, 1, true>(a, st);
  return launch_tile_s<BM, BN, WAVES_M, WAVES_N, GATEUP, NS, OCC, 1, false>(a, st);
}

// Tile shape codes: 256 = 256x256, 192 = 192x256 (one weight set), 160 = 160 token rows x 256 weight rows, 128/129 = 128 x 256,
// 130 = 128x128, 64 = 128x64 (the last two also with the K of a down projection cut into parts, whose fp32
// sums a second kernel adds in order, when the caller provides room for them); 0 = choose from layer-wide
// sizes only (never from the block bounds).
//
// One weight set on a known number of rows (the shared expert): the shape with the least estimated
// time.  A launch takes ceil(items / CUs) rounds of one tile each, a tile costs rows x columns x K
// times a per-shape factor (smaller tiles move more bytes per flop through LDS).  The factors come
// from timing the six shapes at T = 128 ... 16384 on the Qwen shape; the K cut pays a reduction
// pass over its fp32 partial sums (5 us and their bytes, written and read, at 5 TB/s).  What the choice is
// about is filling the chip in whole rounds: gate/up at T = 777 is 176 tiles of 256 rows or 220 of 160 (58 and
// 46 us), the down projection there 112 tiles of 128x128 or twice as many of half the K (44 and 29 us), at
// T = 512 64 tiles or 256 quarters (42 and 25 us); 192 rows: gate/up at T = 2048 484 tiles, two rounds (100 -> 94 us), at 3000
// 152 -> 136, the down projection at 6000 256 tiles (125 -> 115).
static int largest_ksplit(int Kdim) { return Kdim % 512 == 0 ? 8 : Kdim % 256 == 0 ? 4 : Kdim % 128 == 0 ? 2 : 1; }
int tile_down_ksplit(int Kdim) { return largest_ksplit(Kdim); }
struct TileChoice { int code, parts; double cost; };   // (cost: of one weight set, as estimated)
constexpr int NARROW_160 = 1601, NARROW_256 = 2561;   // 160x128 and 256x128: only launched in place of the wider ones (pick_tile)
constexpr double UNITS_PER_US = 3.0e6;   // 256x256x2048 tile: 45 us (a gate/up tile, which counts the columns of one branch, takes twice as long)
static TileChoice pick_tile_shape(int rows, int N, int Kdim, bool gateup, int parts_max, bool leave_room) {
  struct Cand { int code, bm, nout; double c; bool cut; };
  const Cand cands[6] = {{256, 256, gateup ? 128 : 256, 1.0, false}, {192, 192, gateup ? 128 : 256, 1.03, false},
                         {160, 160, gateup ? 128 : 256, 1.07, false},
                         {129, 128, gateup ? 128 : 256, 1.1, false}, {130, 128, gateup ? 64 : 128, 1.42, true},
                         {64, 128, gateup ? 32 : 64, 1.77, true}};
  const double cus = (double)num_cus();
  TileChoice best{129, 1, 0.0};
  for (const Cand& k : cands) {
    // 192x256 leaves other kernels 86 registers of a SIMD and 45 KB of LDS.  256x256, two waves of 210 registers per SIMD and
    // 128 KB, slows them down (16 384 tokens, each kernel's time: row sort 152 -> 243 us, gate logits 45 -> 67), but its own
    // time outweighs that: layers of H 2048, 60 experts, Is 5632 beside gating and sort, us, without it -> with it: 4096 tokens
    // 700 -> 682 (skewed, captured 677 -> 665), 8192 1254 -> 1214, 12 000 skewed 1783 -> 1722, 16 384 2355 -> 2269; 32 experts of
    // H 2560, Is 4096 at 12 000 1964 -> 1903; where it is not picked, and at 3000 and 6000, equal.
    if (k.bm == 192 && leave_room) continue;
    const int most = gateup || !k.cut ? 1 : std::max(1, std::min(parts_max, largest_ksplit(Kdim)));
    for (int parts = 1; parts <= most; parts *= 2) {
      if (k.code == 64 && !gateup && parts == 1) continue;   // (128x128 serves such a batch better)
      const double items = (double)((rows + k.bm - 1) / k.bm) * (double)((N + k.nout - 1) / k.nout) * parts;
      const double rounds = (double)(long)((items + cus - 1) / cus);
      // 160x256 leaves registers but no LDS beside it: the small kernels of the other stream wait for it, which a launch of
      // many rounds must not make them (16 384 tokens: the row sort waited 750 us behind it; layer 2417 us, without 2362)
      if (k.code == 160 && leave_room && rounds > 2.0) continue;
      double cost = rounds * k.bm * k.nout * ((double)Kdim / parts) * k.c;
      if (parts > 1) cost += (5.0 + (double)rows * N * parts * 8.0 / 5.0e6) * UNITS_PER_US;
      if (best.cost == 0.0 || cost < best.cost) best = TileChoice{k.code, parts, cost};
    }
  }
  return best;
}

// Routed experts: the row counts are known only on the device, so the tile height comes from the
// layer-wide mean (never from the block bounds).  An expert near the upper end of the expected
// spread (mean + 1.5 sqrt(mean) rows, the binomial spread of uniform routing) should fit its tiles
// with the least padded work: candidates 128, 160 and 256 rows, each row of a tile costing 1.41,
// 1.23 and 1.0 (smaller tiles move more panel bytes per flop; factors fitted at T = 8192).
// Measured on uniform routing at T = 768 ... 8192 the pick is the fastest shape or within 3 % of
// it; Zipf-skewed routing (mean 273, median 130) and the multi-tenant batch (mean 137) also run
// fastest on its choice (160).
static TileChoice pick_layer_tile(const GemmArgs& a, int tile_rows, bool gateup) {
  if (tile_rows == 64 && !gateup && a.parts_max > 0) return TileChoice{64, std::min(a.parts_max, largest_ksplit(a.Kdim)), 0.0};
  if (tile_rows != 0) return TileChoice{tile_rows, 1, 0.0};
  if (a.offsets == nullptr) return pick_tile_shape(a.rows_total, a.N, a.Kdim, gateup, a.parts_max, a.leave_room != 0);
  const double m = (double)a.mean_rows + 1.5 * sqrt((double)a.mean_rows);
  const int heights[3] = {129, 160, 256};
  const double factor[3] = {1.41, 1.23, 1.0};
  int best = 129;
  double best_cost = 0.0;
  for (int i = 0; i < 3; ++i) {
    const int bm = heights[i] == 129 ? 128 : heights[i];
    const double cost = ceil(m / bm) * bm * factor[i];
    if (best_cost == 0.0 || cost < best_cost) { best_cost = cost; best = heights[i]; }
  }
  // Layers with few experts: fewer than two rounds of the chip with that height (the whole layer's tiles, not the
  // block's).  Then whole rounds count, and narrower tiles that give every CU one: cost = rounds x rows x columns x
  // factor (the factors above; 1.82 and 2.26 for 128x128 and 128x64).  Down projection, us, before -> now: 8 experts of
  // H 4096, I 7168 at 34 rows 117 -> 76 (128x256 was 128 tiles), at 200 rows 186 -> 128, 4 of H 2048, I 2560 at 60 rows
  // 44 -> 23, 8 of H 2048, I 8192 at 40 rows 101 -> 53; gate/up 4 of H 2048, I 2560 at 34 rows 35 -> 26.
  // (A call that also hosts the shared experts picks the same, so that its routed rows keep the bits of the plain call.)
  // With two rounds
  // and more the heights' rule is the better one (8 experts of H 4096 at 1000 rows, gate/up: 903 us as picked, 938 and
  // 926 with 128 and 160 rows).
  const long cus = num_cus();
  auto items_of = [&](int bm, int nout) -> double {
    return (double)a.experts_layer * ceil(m / bm) * (double)((a.N + nout - 1) / nout);
  };
  const int wide = gateup ? 128 : 256;
  if (a.experts_layer > 0 && items_of(best == 129 ? 128 : best, wide) < 2.0 * (double)cus) {
    struct Cand { int code, bm, bn; double c; };
    const Cand cands[5] = {{256, 256, 256, 1.0}, {160, 160, 256, 1.23}, {129, 128, 256, 1.41}, {130, 128, 128, 1.82}, {64, 128, 64, 2.26}};
    best_cost = 0.0;
    for (const Cand& k : cands) {
      const double cost = ceil(items_of(k.bm, gateup ? k.bn / 2 : k.bn) / (double)cus) * k.bm * k.bn * k.c;
      if (best_cost == 0.0 || cost < best_cost) { best_cost = cost; best = k.code; }
    }
  }
  return TileChoice{best, 1, 0.0};
}
// What a call launches for the layer's tile shape.  A call on a block of a few experts can have fewer tiles than the chip
// has compute units; narrower tiles of the same height then give more of them work.  Every output element is summed in the
// same order whatever the tile's columns (the K start of a single-tile expert goes by the columns of the layer's shape), so
// the bits stay those of the uncut layer.  cost = rounds x columns x factor (a step of a tile of half the columns takes
// more than half the time), the rounds counted for even routing and, weighing more, for skewed routing: with a mean of r
// tiles of rows, experts then take 1 + 1.15 (r - 0.3) tiles on average (r + 0.8 beyond one; four tenants with normal router
// biases, 700 to 3000 tokens).  The skew decides close cases: 15 experts of 137 rows even are 120 tiles of the down
// projection, 240 half ones take 27 instead of 34 us, but skewed they are 152-192 and the half ones take two rounds.  What
// wins by less than a tenth is left alone (16 of 64 experts of H 1536, I 1024 at 84 rows, 128x64 for 128x128: 3 us more).
// us, one call per block, 256 -> narrower: 60 experts of H 2048, I 1408 in blocks of 7 at 137 rows 41+31 -> 32+23, of 15
// at 200 rows 69+47 -> 61+31, at 52 rows 39+28 -> 39+22; 16 of H 3072, I 4096 at 100 rows in blocks of 4 63+58 -> 46+36,
// of 2 54+56 -> 32+31; 8 of H 4096, I 7168 in blocks of 2 at 60 rows 61+62 -> 45+45, at 250 rows 88+103 -> 88+76.
// The line was fitted to the tenants' routing; against the build without the rule (and a few other changes worth 1 to 2 %)
// layers in blocks gain with every other kind that was timed, us, Zipf unless said: 60 experts of H 2048, I 1408 in blocks of
// 7 at 1500 tokens 605 -> 497, at 2048 652 -> 544, of 5 at 6000 1430 -> 1159, of 6 at 3000 (even) 1116 -> 665, of 15 at 600 to 3000
// 287 -> 275, 321 -> 314, 404 -> 396, 559 -> 501; 64 of H 1536, I 1024 in blocks of 8 at 3000 590 -> 563, of 16 at 900 252 ->
// 246; 32 of H 2560, I 1536 in blocks of 8 at 1500 545 -> 456; 8 of H 4096, I 7168 in blocks of 2 at 1000 836 -> 768; 16 of H
// 3072, I 4096 in blocks of 4 at 600 746 -> 537.
static int tile_columns(int code, bool gateup) {
  const int bn = code == 64 ? 64 : code == 130 || code == NARROW_160 || code == NARROW_256 ? 128 : 256;
  return gateup ? bn / 2 : bn;
}
static TileChoice pick_tile(GemmArgs& a, int tile_rows, bool gateup) {
  TileChoice c = pick_layer_tile(a, tile_rows, gateup);
  a.rot_shift = __builtin_ctz(tile_columns(c.code, gateup));
  if (tile_rows != 0 || a.offsets == nullptr || a.n_shared > 0) return c;
  const int layer = c.code;
  const int f = layer == 256 ? 0 : layer == 160 ? 1 : 2;
  const int family[3][3] = {{256, NARROW_256, 0}, {160, NARROW_160, 0}, {129, 130, 64}};
  const double factor[3] = {1.0, 1.29, 1.75};
  const int heights[3] = {256, 160, 128};
  const double r = (double)a.mean_rows / heights[f], cus = (double)num_cus();
  const double even = ceil(((double)a.mean_rows + 1.5 * sqrt((double)a.mean_rows)) / heights[f]);
  const double skewed = r < 0.3 ? 1.0 : r < 1.0 ? 1.0 + 1.15 * (r - 0.3) : r + 0.8;
  double best = 0.0;
  for (int i = 0; i < 3 && family[f][i] != 0; ++i) {
    const int nout = tile_columns(family[f][i], gateup);
    if (nout > tile_columns(layer, gateup)) continue;
    const double per_row_tile = (double)(a.hi - a.lo) * (double)((a.N + nout - 1) / nout);
    const double cost = (ceil(per_row_tile * even / cus) + 2.0 * ceil(per_row_tile * skewed / cus)) * nout * factor[i];
    if (best == 0.0 || cost < 0.9 * best) { best = cost; c.code = family[f][i]; }
  }
  return c;
}
// The shared expert's gate/up tiles in the launch of the routed experts': both contract over H, so they are alike, and the
// walk draws them alternately.  What it saves is rounds that are not full (2048 tokens of H 2048, 60 experts of I 1408, top
// 4, Is 5632: 660 tiles run as three rounds and 484 as two; together 1232 of 160 rows as five) and tiles that wait for weights
// while nothing multiplies.  us, two launches -> one: 777 tokens 175 -> 162, 1400 210 -> 193, 2048 252 -> 219 (with skewed
// routing 256 -> 262), 3000 327 -> 299, 4096 426 -> 396 (skewed 416 -> 401), 8192 765 -> 744; a whole layer at
// 2048 skewed tokens 458 -> 442, with four tenants 468 -> 442.  The down projections stay apart:
// their contractions differ (22 and 88 K steps), and the shared expert cut into sets gains nothing (136 -> 132 at 2048).
// Only with full-width tiles: layers of few or small experts and calls on a few of them take narrower ones, which the shared
// expert's many rows do not want; only with more tokens than a tile has rows, for the K start of single tiles is not the shared expert's; only
// where the rounds that its tiles add cost no more than its own launch in the shape that it takes there (both in the units
// and factors of pick_tile_shape), and about 6 us for the launch: with even routing, and as a share of a round per tile, for
// skewed routing fills the last round differently.  Counted are all column tiles of all sets: one past the columns of a
// narrower last set walks K like any other and stores nothing.  A layer in us, apart -> in one launch: 60 experts of H 2048, I
// 1152, Is 1216 at 2100 tokens, half of whose shared tiles hold columns, 330 -> 322; what the line keeps apart: 16 of H 1024, I
// 4096, Is 192 at 4513 (58 of 928 tiles hold columns) 233 -> 279, 48 of H 1024, I 4032, Is 512 at 9015 437 -> 543, 64 of H
// 1536, I 1024 at 66 rows (two full rounds, and 0.4 of Is 2048) 195 -> 200.  Near the line both cost the same: 32 of H 1024, I
// 2048, Is 8192 at 4007 344 -> 352 on one card, 362 -> 361 on another, 32 of H 1024, I 960, Is 1984 at 6000 351 -> 347 and 364 -> 368.
bool tile_hosts_shared(const GemmArgs& a, int tokens, int Is) {
  GemmArgs apart = a;
  const int code = pick_tile(apart, 0, true).code;
  if (code != 256 && code != 160 && code != 129) return false;
  const int sets = (Is + a.N - 1) / a.N, columns = (a.N + 127) / 128;      // sets, and column tiles of one
  if (tokens <= 256 || a.hi - a.lo + sets > TILE_EMAX) return false;
  const double bm = code == 129 ? 128.0 : code, cus = (double)num_cus(), factor = code == 256 ? 1.0 : code == 160 ? 1.07 : 1.1;
  const double m = (double)a.mean_rows + 1.5 * sqrt((double)a.mean_rows);
  const double routed = (double)(a.hi - a.lo) * ceil(m / bm) * (double)columns;
  const double shared = ceil(tokens / bm) * (double)(sets * columns);
  const double rounds = std::max(ceil((routed + shared) / cus) - ceil(routed / cus), shared / cus);
  return rounds * bm * 128.0 * (double)a.Kdim * factor <= pick_tile_shape(tokens, Is, a.Kdim, true, 0, false).cost + 3.0 * UNITS_PER_US;
}
int launch_tile_gateup(const GemmArgs& layer, int tile_rows, hipStream_t st) {
  GemmArgs a = layer;
  const int t = pick_tile(a, tile_rows, true).code;
  if (t == NARROW_160) return launch_tile_t<160, 128, 1, 4, true, 4, 1>(a, st);
  if (t == NARROW_256) return launch_tile_t<256, 128, 2, 2, true, 3, 1>(a, st);
  if (t == 64) return launch_tile_t<128, 64, 4, 1, true, 6, 1>(a, st);
  if (t == 130) return launch_tile_t<128, 128, 2, 2, true, 4, 1>(a, st);
  if (t >= 256) return launch_tile_t<256, 256, 2, 4, true, 2, 1>(a, st);
  if (t == 192) return launch_tile_s<192, 256, 2, 2, true, 2, 1, 1, false>(a, st);   // (one weight set only)
  if (t == 160) return launch_tile_t<160, 256, 1, 4, true, 3, 1>(a, st);
  return launch_tile_t<128, 256, 1, 4, true, 3, 1>(a, st);
}
// A down projection in tiles of 128 token rows by BN, whole or in K parts (side by side in a.Cpart, or in turn)
template <int BN, int WAVES_M, int WAVES_N, int NS>
static int launch_tile_cut(const GemmArgs& a, int parts, bool in_turn, hipStream_t st) {
  switch (parts) {
    case 8:
      return in_turn ? launch_tile_s<128, BN, WAVES_M, WAVES_N, false, NS, 1, 8, false, true>(a, st)
                     : launch_tile_s<128, BN, WAVES_M, WAVES_N, false, NS, 1, 8, false>(a, st);
    case 4:
      return in_turn ? launch_tile_s<128, BN, WAVES_M, WAVES_N, false, NS, 1, 4, false, true>(a, st)
                     : launch_tile_s<128, BN, WAVES_M, WAVES_N, false, NS, 1, 4, false>(a, st);
    case 2:
      return in_turn ? launch_tile_s<128, BN, WAVES_M, WAVES_N, false, NS, 1, 2, false, true>(a, st)
                     : launch_tile_s<128, BN, WAVES_M, WAVES_N, false, NS, 1, 2, false>(a, st);
    default: return launch_tile_t<128, BN, WAVES_M, WAVES_N, false, NS, 1>(a, st);
  }
}
// *parts: in how many K parts the output was left in a.Cpart (1: the output itself is written)
int launch_tile_down(const GemmArgs& layer, int tile_rows, hipStream_t st, int* parts) {
  GemmArgs a = layer;
  const TileChoice c = pick_tile(a, tile_rows, false);
  const int t = c.code;
  const bool in_turn = c.parts > std::max(1, a.parts_room);
  *parts = in_turn ? 1 : c.parts;
  if (t == NARROW_160) return launch_tile_t<160, 128, 1, 4, false, 4, 1>(a, st);
  if (t == NARROW_256) return launch_tile_t<256, 128, 2, 2, false, 3, 1>(a, st);
  if (t == 64) return launch_tile_cut<64, 4, 1, 6>(a, c.parts, in_turn, st);   // (without parts: whole K per tile)
  if (t == 130) return launch_tile_cut<128, 2, 2, 4>(a, c.parts, in_turn, st);
  if (t >= 256) return launch_tile_t<256, 256, 2, 4, false, 2, 1>(a, st);
  if (t == 192) return launch_tile_s<192, 256, 2, 2, false, 2, 1, 1, false>(a, st);
  if (t == 160) return launch_tile_t<160, 256, 1, 4, false, 3, 1>(a, st);
  return launch_tile_t<128, 256, 1, 4, false, 3, 1>(a, st);
}

}  // namespace moe
