// C entry points of the MoE-layer library: argument checks and the choice of kernel shapes.
// Semantics of every call are stated in include/moe.h.
#include <algorithm>
#include <atomic>
#include "../../include/moe.h"
#include "../../include/moe_tuning.h"
#include "common.h"

using namespace moe;

namespace {

size_t align256(size_t n) { return (n + 255) & ~(size_t)255; }

// No byte of [a, a + na) in [b, b + nb)
bool apart(const void* a, size_t na, const void* b, size_t nb) {
  const uintptr_t p = (uintptr_t)a, q = (uintptr_t)b;
  return na == 0 || nb == 0 || (p < q ? q - p >= na : p - q >= nb);
}

bool dims_ok(int H) { return H > 0 && H % 64 == 0; }

// Shared expert: most parts of its down projection along K, for which the workspace helper reports room: 8 up to 512
// tokens, beyond that as many (a power of two) as it takes 128x128 tiles to 256 items, one round of the chip (the compute
// units of the MI355X: the helper answers without a device).
constexpr int SHARED_SMALL_T = 512;
constexpr int SHARED_KPARTS_MAX = 8;
int shared_parts_room(int T, int H) {
  if (T <= SHARED_SMALL_T) return SHARED_KPARTS_MAX;
  const long tiles = ((long)T + 127) / 128 * (((long)H + 127) / 128);
  int parts = 1;
  while (parts < SHARED_KPARTS_MAX && 2 * parts * tiles <= 256) parts *= 2;
  return parts > 1 ? parts : 0;
}

// Tokens up to which the streaming kernel serves the shared expert, riding along with the routed ones or by itself, and
// the K parts of its down projection there: up to four of eight K steps and more, then parts of 22.  (A layer of H 2048,
// Is 5632: four parts, with eight it takes about 2 us more at 1 to 24 tokens; 12 experts of H 1024 and Is 1536 at 24
// tokens: 32 us in three parts, 38 in one.)  Both depend on the shared expert's own sizes alone: its bits are the same in
// every sequence of calls.  (More figures beside that kernel.)
constexpr int SHARED_FEW_T = 32;
int shared_few_parts(int Is) { return std::max({1, std::min(4, Is / 512), std::min(SHARED_KPARTS_MAX, Is / 1408)}); }

// Tokens up to which the streaming kernels take the sets of a block call that hosts the shared experts along: four passes
// of the narrow one, two of the wide one.  A layer in us, taken along | in tiles of their own | before routed rows of
// these sizes were streamed (all in tiles): 12 experts of H 1024, I 768, Is 1536 at 20 tokens, top 4 36 | 56 | 44, at 36,
// top 2 34 | 50 | 44, at 150 43 | 63 | 51; 15 of H 2048, I 512, Is 2048, top 1 at 60 tokens 52 | 60 | 65, at 90 (narrow)
// 62 | 61 | 68; 8 of H 2560, I and Is 4096, top 1 at 200 (wide, three passes) 165 | 158 | 183.  What stays slower than all
// in tiles: 27 to 32 rows per expert with more tokens than that (60 experts of H 2048 at T = 470 284 against 274, 15 at 400
// 78 against 71), for the routed rows must keep the bits of the plain block call, whose layer is the faster one for it
// (284 against 307, 78 against 110).
constexpr int FUSED_NARROW_T = 64, FUSED_WIDE_T = 192;

// Which kernels serve an FFN with `mean_rows` expected rows per expert.  The choice uses only
// layer-wide sizes (never the block bounds), so a row's result does not depend on the block cut.
// policy: 0 = automatic; 3 and 5 = MFMA tiles of 128 token rows by 256 weight rows; 4 = 256 by 256;
//         8 = 128 by 64, the down projection cut along K (few rows in all, one weight set);
//         9 = weight streaming through wave-private LDS rings (few rows per expert);
//         10 = 128 by 128; 11 = 160 by 256.  Any other number is refused.
// Bits 8 and 9 of the policy word restrict a call to one of its two kernels (0x100: gate/up
// only, 0x200: down projection only), so that each can be timed on its own.  Bit 10 (0x400, shared
// expert with automatic shapes): its first kernel takes no tile shape that keeps small kernels of
// other streams (gating, micro-batch construction) off the CUs for long (pick_tile_shape says which).
struct Plan { bool valid; bool stream; int tile_rows; bool do_gateup; bool do_down; };
Plan make_plan(int mean_rows, int n_experts_layer, int policy_word) {
  Plan p{};
  const int phase = (policy_word >> 8) & 3;
  const int policy = policy_word & 0xff;
  p.valid = (policy_word & ~0x7ff) == 0;
  p.do_gateup = phase == 0 || (phase & 1);
  p.do_down = phase == 0 || (phase & 2);
  switch (policy) {
    case 0: break;
    case 3: p.tile_rows = 128; return p;
    case 4: p.tile_rows = 256; return p;
    case 5: p.tile_rows = 129; return p;
    case 8: p.tile_rows = 64; return p;
    case 9: p.stream = true; return p;
    case 10: p.tile_rows = 130; return p;
    case 11: p.tile_rows = 160; return p;
    default: p.valid = false; return p;
  }
  // One weight set on all rows (the shared expert): MFMA tiles whose shape each kernel picks from
  // its tile count (pick_tile_shape).  Routed experts: weight streaming up to a mean of 32 rows per
  // expert, the MFMA tiles beyond (their height picked from the layer-wide mean).  Measured with cold
  // caches, gate/up + down in us, streaming against tiles: 60 experts of H 2048, I 1408 at 26 rows 125 + 66
  // and 135 + 69, at 34 rows 134 + 72 and 137 + 72; 128 of H 1024, I 768 at 31 rows 79 + 45 and 83 + 48;
  // 8 of H 4096, I 7168 at 5 rows 157 + 77 and 164 + 112, at 30 rows 179 + 83 and 166 + 117.
  p.stream = n_experts_layer > 1 && mean_rows <= 32;
  p.tile_rows = 0;
  return p;
}

// *parts: K parts in which the down projection was left in dn.Cpart (1: its output is complete)
int ffn_forward(const GemmArgs& gu, const GemmArgs& dn, const Plan& p, hipStream_t st, int* parts) {
  int rc = 0;
  *parts = 1;
  if (p.stream) {
    if (p.do_gateup && (rc = launch_stream_lds_gateup(gu, st)) != 0) return rc;
    if (p.do_down) rc = launch_stream_lds_down(dn, st);
    return rc;
  }
  if (p.do_gateup && (rc = launch_tile_gateup(gu, p.tile_rows, st)) != 0) return rc;
  if (p.do_down) rc = launch_tile_down(dn, p.tile_rows, st, parts);
  return rc;
}

void set_shared_parts(GemmArgs& dn, int parts, int Is) {
  dn.shared_parts = parts;
  dn.part_steps = Is / 64 / parts;
  dn.part_extra = Is / 64 % parts;
}

// The shared expert riding along with the routed experts of a few tokens (see expert_stream_lds.hip): `sets` sets of I
// columns of its hidden layer h [T,Is], and its output as `parts` fp32 parts [T,H].
struct Riders { const void *x, *Wsg, *Wsu, *Wsd; void* h; float* part; int sets, parts, T, Is; };

// The shared expert's gate/up tiles in the launch of the routed experts' (see expert_tile.hip): h is its hidden layer [T,Is].
struct Hosted { const void *x, *Wsg, *Wsu; void* h; int T, Is; };

// The micro-batch of a layer with few pairs, constructed inside the first launch of its experts (see expert_stream_lds.hip)
struct Sort { const int32_t* ids; int32_t *offsets, *src, *rows; void* Xp; };
// What it costs is the look at the ids of every wave of that launch (`experts` of them by 16 columns each): of those without
// rows, which otherwise leave after two scalar loads, while few others run (the first line), and of those with rows, whose
// number grows with the pairs too (the second).  A layer in us, sorted apart -> here, on both sides of the first: 256 experts
// of H 2048 at 8 pairs, I 768 47.0 -> 45.3, I 1024 50.9 -> 49.7 and 49.9 -> 49.8, I 1408 57.3 -> 57.8, I 2048 67.1 -> 69.7, at 16 92.4 ->
// 93.1, at 32 146 -> 143; 60 of I 1408 at 4 47 -> 43; 160 of H 1024, I 2560 at 6 43.3 -> 44.2, 64 of I 4096 at 4 42.0 -> 43.5, 256 of
// I 4096 at 16 94 -> 104.  Of the second: 256 experts of H 2048, I 768 at 64 pairs 112 -> 110, at 96 148 -> 149, at 128 178 ->
// 183; of H 1024, I 512 at 72 54.3 -> 52.3, at 128 75.1 -> 77.3; I 256 at 128 56.9 -> 52.7; 160 of I 1536 at 60 92.9 -> 91.3, at 96
// 122.0 -> 123.8; 64 of I 1536 at 72 81.6 -> 79.1, at 128 100.9 -> 101.8; 128 of I 1408 at 72 95.4 -> 93.7, of I 512 at 128 59.1 ->
// 57.8.
bool sort_in_gateup(int P, int H, int E, int I, int experts) {
  const int mean_rows = (P + E - 1) / E;
  const long long waves = (long long)experts * ((I + 15) / 16);
  return P <= SORT_HERE_MAX && waves < 2048ll * std::max(P, 6) && waves * P * P <= 90000000ll && E > 1 &&
         make_plan(mean_rows, E, 0).stream && stream_narrow(mean_rows, H);
}

int expert_group_forward_impl(int group_lo, int group_hi, const int32_t* ids, const void* A, const int32_t* gather,
                              int gather_div,
                              const int32_t* expert_offsets, const void* Wg, const void* Wu, const void* Wd, int P,
                              int H, int E, int I, void* Yp, void* workspace, size_t workspace_bytes, int policy,
                              void* stream, const Riders* riders = nullptr, const Sort* sort = nullptr, const Hosted* hosted = nullptr,
                              bool* is_hosted = nullptr) {
  if (P < 0 || !dims_ok(H) || !dims_ok(I) || E < 1 || E > 256) return MOE_ERR_SHAPE;
  if (group_lo < 0 || group_hi > E || group_lo >= group_hi) return MOE_ERR_SHAPE;
  if ((long long)P * (H > I ? H : I) >= (1ll << 31)) return MOE_ERR_SHAPE;
  if (P == 0) return MOE_OK;
  if (!A || !expert_offsets || !Wg || !Wu || !Wd || !Yp || !workspace) return MOE_ERR_NULL;
  if (workspace_bytes < (size_t)P * (size_t)I * 2) return MOE_ERR_WORKSPACE;   // h, bf16 [P,I]
  const int mean_rows = (P + E - 1) / E;
  const Plan plan = make_plan(mean_rows, E, policy);
  if (!plan.valid) return MOE_ERR_SHAPE;
  if (riders != nullptr && (!plan.stream || mean_rows > STREAM_FEW_ROWS)) return MOE_ERR_SHAPE;
  GemmArgs gu{};
  gu.A = (const bf16_t*)A; gu.B0 = (const bf16_t*)Wg; gu.B1 = (const bf16_t*)Wu; gu.C = (bf16_t*)workspace;
  gu.offsets = expert_offsets; gu.lo = group_lo; gu.hi = group_hi; gu.ids = ids; gu.rows_fixed = 0; gu.rows_total = P;
  gu.mean_rows = mean_rows; gu.experts_layer = E; gu.N = I; gu.Kdim = H;
  GemmArgs dn = gu;
  gu.gather = gather; gu.gather_div = gather_div;   // only the first kernel reads token rows
  dn.A = (const bf16_t*)workspace; dn.B0 = (const bf16_t*)Wd; dn.B1 = nullptr; dn.C = (bf16_t*)Yp;
  dn.N = H; dn.Kdim = I;
  if (sort != nullptr) {
    gu.sort_ids = sort->ids; gu.n_pairs = P; gu.sort_offsets = sort->offsets; gu.sort_src = sort->src; gu.sort_rows = sort->rows;
    gu.sort_copy = (bf16_t*)sort->Xp;
  }
  if (riders != nullptr) {
    gu.n_shared = riders->sets;
    dn.n_shared = riders->parts;
    set_shared_parts(dn, riders->parts, riders->Is);
    gu.shared_rows = dn.shared_rows = riders->T;
    gu.ldb_shared = dn.ldb_shared = riders->Is;
    gu.As = (const bf16_t*)riders->x; gu.Bs0 = (const bf16_t*)riders->Wsg; gu.Bs1 = (const bf16_t*)riders->Wsu;
    gu.Cs = (bf16_t*)riders->h;
    dn.As = (const bf16_t*)riders->h; dn.Bs0 = (const bf16_t*)riders->Wsd; dn.Cpart = riders->part;
  }
  if (hosted != nullptr && !plan.stream && tile_hosts_shared(gu, hosted->T, hosted->Is)) {
    gu.n_shared = (hosted->Is + I - 1) / I;
    gu.shared_rows = hosted->T;
    gu.rows_routed = P;
    gu.rows_total = P + gu.n_shared * hosted->T;
    gu.Bs0 = (const bf16_t*)hosted->Wsg; gu.Bs1 = (const bf16_t*)hosted->Wsu;
    gu.shared_b_step = (long)I * H;
    gu.ldb_shared = H;
    gu.As = (const bf16_t*)hosted->x;
    gu.Cs = (bf16_t*)hosted->h;
    gu.shared_cols = hosted->Is;
    *is_hosted = true;
  }
  int parts;   // (no Cpart of its own: always 1)
  return ffn_forward(gu, dn, plan, (hipStream_t)stream, &parts);
}
}  // namespace

// Scratch memory of moe_permute_static: the per-chunk expert histogram of the counting sort, which
// moe_permute keeps in the caller's workspace.  Every GPU the library runs on holds its own copy of
// the array at its own address until the process ends.  In host code the array's name is not a
// device address: the address on the current device is asked for once per device
// (hipGetSymbolAddress) and kept; only that pointer is handed to kernels.
static __device__ __align__(256) unsigned char scratch[MOE_PERMUTE_STATIC_SCRATCH_BYTES];
static std::atomic<void*> scratch_on_device[64];   // by device id

static int static_scratch(void** out) {
  int dev = -1;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return MOE_ERR_LAUNCH;
  void* p = scratch_on_device[dev].load(std::memory_order_acquire);
  if (p == nullptr) {
    if (hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)) != hipSuccess || p == nullptr) return MOE_ERR_LAUNCH;
    scratch_on_device[dev].store(p, std::memory_order_release);
  }
  *out = p;
  return MOE_OK;
}

#ifndef MOE_BUILD_ID
#define MOE_BUILD_ID "unstamped"
#endif

extern "C" {

const char* moe_build_id(void) { return MOE_BUILD_ID; }

int moe_tile_clock_buffer(int64_t* clocks, int workgroups) {
  if (clocks != nullptr && workgroups < 1) return MOE_ERR_SHAPE;
  moe::set_tile_clock_buffer(reinterpret_cast<long long*>(clocks), clocks == nullptr ? 0 : workgroups);
  return MOE_OK;
}

int moe_probe_mfma(const void* operands, size_t operand_bytes, int iters, int workgroups, int64_t* clocks, void* stream) {
  if (operands == nullptr || clocks == nullptr) return MOE_ERR_NULL;
  if (operand_bytes < MOE_PROBE_OPERAND_BYTES || iters < 1 || iters > (1 << 20) || workgroups < 1 || workgroups > 65535)
    return MOE_ERR_SHAPE;
  return moe::launch_mfma_probe(operands, iters, workgroups, reinterpret_cast<long long*>(clocks), (hipStream_t)stream) == 0
             ? MOE_OK : MOE_ERR_LAUNCH;
}

const char* moe_status_string(int status) {
  switch (status) {
    case MOE_OK: return "ok";
    case MOE_ERR_NULL: return "a required pointer is NULL";
    case MOE_ERR_SHAPE: return "a size or an expert range is outside the supported limits";
    case MOE_ERR_WORKSPACE: return "workspace too small";
    case MOE_ERR_LAUNCH: return "kernel launch failed";
    default: return "unknown status";
  }
}

size_t moe_permute_workspace_bytes(int T, int K, int E) {
  if (T <= 0 || K <= 0 || E <= 0) return 0;
  const size_t chunks = ((size_t)T * (size_t)K + 63) / 64;   // pairs of each expert per 64-pair chunk
  return align256(chunks * (size_t)E * 4);
}
size_t moe_expert_workspace_bytes(int P, int I) {
  if (P <= 0 || I <= 0) return 0;
  return align256((size_t)P * (size_t)I * 2);
}
// h [T,Is] bf16, then (batches that leave CUs idle otherwise) the fp32 partial outputs of a down projection cut along K
size_t moe_shared_workspace_bytes(int T, int H, int Is) {
  if (T <= 0 || H <= 0 || Is <= 0) return 0;
  size_t n = align256((size_t)T * (size_t)Is * 2);
  n += (size_t)shared_parts_room(T, H) * (size_t)T * (size_t)H * 4;
  return n;
}
size_t moe_workspace_bytes(int T, int H, int E, int K, int I, int Is) {
  size_t a = moe_permute_workspace_bytes(T, K, E);
  size_t b = moe_expert_workspace_bytes(T * K, I);
  size_t c = moe_shared_workspace_bytes(T, H, Is);
  size_t m = a > b ? a : b;
  return m > c ? m : c;
}

int moe_route(const void* x, const void* Wr, const float* bias, int T, int H, int E, int K, int renorm,
              int32_t* topk_ids, float* topk_w, void* stream) {
  if (T < 0 || !dims_ok(H) || H > 8192 || E < 1 || E > 256 || K < 1 || K > 16 || K > E) return MOE_ERR_SHAPE;
  if (T == 0) return MOE_OK;
  if (!x || !Wr || !topk_ids || !topk_w) return MOE_ERR_NULL;
  return launch_route(x, Wr, bias, nullptr, 0, T, H, E, K, renorm, topk_ids, topk_w, (hipStream_t)stream);
}

int moe_route_segments(const void* x, const void* Wr, const float* bias_rows, const int32_t* seg_offsets, int n_seg,
                       int T, int H, int E, int K, int renorm, int32_t* topk_ids, float* topk_w, void* stream) {
  if (T < 0 || !dims_ok(H) || H > 8192 || E < 1 || E > 256 || K < 1 || K > 16 || K > E) return MOE_ERR_SHAPE;
  if (n_seg < 1 || n_seg > 4096) return MOE_ERR_SHAPE;
  if (T == 0) return MOE_OK;
  if (!x || !Wr || !bias_rows || !seg_offsets || !topk_ids || !topk_w) return MOE_ERR_NULL;
  return launch_route(x, Wr, bias_rows, seg_offsets, n_seg, T, H, E, K, renorm, topk_ids, topk_w,
                      (hipStream_t)stream);
}

static int permute_refusal(const int32_t* topk_ids, const void* x, int T, int H, int E, int K, const int32_t* expert_offsets,
                           const int32_t* src_of_row, const int32_t* row_of_pair, const void* Xp, const void* workspace,
                           size_t workspace_bytes) {
  if (T < 0 || !dims_ok(H) || E < 1 || E > 256 || K < 1 || K > 16 || K > E) return MOE_ERR_SHAPE;
  if ((long long)T * K * H >= (1ll << 31)) return MOE_ERR_SHAPE;
  if (!expert_offsets) return MOE_ERR_NULL;
  if (T > 0 && (!topk_ids || !src_of_row || !row_of_pair || !workspace)) return MOE_ERR_NULL;
  if (T > 0 && Xp && !x) return MOE_ERR_NULL;   // Xp == NULL: index arrays only, x is not read
  if (T > 0 && workspace_bytes < (((size_t)T * K + 63) / 64) * (size_t)E * 4) return MOE_ERR_WORKSPACE;
  return MOE_OK;
}

int moe_permute(const int32_t* topk_ids, const void* x, int T, int H, int E, int K, int32_t* expert_offsets,
                int32_t* src_of_row, int32_t* row_of_pair, void* Xp, void* workspace, size_t workspace_bytes,
                void* stream) {
  const int rc = permute_refusal(topk_ids, x, T, H, E, K, expert_offsets, src_of_row, row_of_pair, Xp, workspace, workspace_bytes);
  if (rc != MOE_OK) return rc;
  return launch_permute(topk_ids, x, T, H, E, K, expert_offsets, src_of_row, row_of_pair, Xp, workspace,
                        (hipStream_t)stream);
}

int moe_permute_static(const int32_t* topk_ids, const void* x, int T, int H, int E, int K, int32_t* expert_offsets,
                       int32_t* src_of_row, int32_t* row_of_pair, void* Xp, void* stream) {
  if (T < 0 || !dims_ok(H) || E < 1 || E > 256 || K < 1 || K > 16 || K > E) return MOE_ERR_SHAPE;
  if ((long long)T * K * H >= (1ll << 31)) return MOE_ERR_SHAPE;
  if (!expert_offsets) return MOE_ERR_NULL;
  if (T > 0 && (!topk_ids || !src_of_row || !row_of_pair)) return MOE_ERR_NULL;
  if (T > 0 && Xp && !x) return MOE_ERR_NULL;
  if ((((size_t)T * K + 63) / 64) * (size_t)E * 4 > (size_t)MOE_PERMUTE_STATIC_SCRATCH_BYTES) return MOE_ERR_WORKSPACE;
  void* table = nullptr;
  const int rc = static_scratch(&table);
  if (rc != MOE_OK) return rc;
  // (the histogram kernel writes every table entry it later reads, so what an earlier call left
  // behind needs no clearing)
  return launch_permute(topk_ids, x, T, H, E, K, expert_offsets, src_of_row, row_of_pair, Xp, table,
                        (hipStream_t)stream);
}

int moe_expert_group_forward_ex(int group_lo, int group_hi, const void* Xp, const int32_t* expert_offsets,
                                const void* Wg, const void* Wu, const void* Wd, int P, int H, int E, int I,
                                void* Yp, void* workspace, size_t workspace_bytes, int policy, void* stream) {
  return expert_group_forward_impl(group_lo, group_hi, nullptr, Xp, nullptr, 1, expert_offsets, Wg, Wu, Wd, P, H, E, I, Yp,
                                   workspace, workspace_bytes, policy, stream);
}

int moe_expert_group_forward_gather(int group_lo, int group_hi, const void* x, const int32_t* src_of_row, int K,
                                    const int32_t* expert_offsets, const void* Wg, const void* Wu, const void* Wd,
                                    int P, int H, int E, int I, void* Yp, void* workspace, size_t workspace_bytes,
                                    int policy, void* stream) {
  if (K < 1 || K > 16 || (P > 0 && P % K != 0)) return MOE_ERR_SHAPE;
  if (P > 0 && !src_of_row) return MOE_ERR_NULL;
  return expert_group_forward_impl(group_lo, group_hi, nullptr, x, src_of_row, K, expert_offsets, Wg, Wu, Wd, P, H, E, I,
                                   Yp, workspace, workspace_bytes, policy, stream);
}

int moe_expert_list_forward(const int32_t* expert_ids, int n_ids, const void* tokens, const int32_t* src_of_row, int K,
                            const int32_t* expert_offsets, const void* Wg, const void* Wu, const void* Wd, int P,
                            int H, int E, int I, void* Yp, void* workspace, size_t workspace_bytes, int policy,
                            void* stream) {
  if (n_ids < 1 || n_ids > E) return MOE_ERR_SHAPE;
  if (!expert_ids) return MOE_ERR_NULL;
  if (src_of_row && (K < 1 || K > 16 || (P > 0 && P % K != 0))) return MOE_ERR_SHAPE;
  // positions [0, n_ids) of the list take the place of the id range; the range checks see [0, n_ids)
  return expert_group_forward_impl(0, n_ids, expert_ids, tokens, src_of_row, src_of_row ? K : 1, expert_offsets, Wg, Wu,
                                   Wd, P, H, E, I, Yp, workspace, workspace_bytes, policy, stream);
}

int moe_fused_shared_sets(int T, int H, int E, int K, int I, int Is) {
  if (T <= 0 || K < 1 || E < 1 || I <= 0 || Is <= 0 || !dims_ok(H) || !dims_ok(I) || Is % I != 0) return 0;
  const int ns = Is / I;
  if (ns > MOE_SHARED_SETS_MAX || E + ns > 256) return 0;
  const long long P = (long long)T * K;
  if ((P + (long long)ns * T) * (H > I ? H : I) >= (1ll << 31)) return 0;
  return E < 16 || (P + E - 1) / E > 26 ? ns : 0;     // decode-sized batches of many experts keep the separate calls
}

size_t moe_fused_workspace_bytes(int T, int K, int I, int Is) {
  if (T <= 0 || K <= 0 || I <= 0 || Is <= 0 || Is % I != 0) return 0;
  return align256(((size_t)T * K + (size_t)(Is / I) * T) * (size_t)I * 2);
}

int moe_expert_group_forward_fused(int group_lo, int group_hi, const void* x, const int32_t* src_of_row, int K,
                                   const int32_t* expert_offsets, const void* Wg, const void* Wu, const void* Wd,
                                   const void* Wsg, const void* Wsu, const void* Wsd, const void* wgate, int T, int H,
                                   int E, int I, int Is, void* Yp, void* S_parts, float* sg, void* workspace,
                                   size_t workspace_bytes, int policy, void* stream) {
  if (T < 0 || K < 1 || K > 16 || !dims_ok(H) || !dims_ok(I) || E < 1 || E > 256) return MOE_ERR_SHAPE;
  if (group_lo < 0 || group_hi > E || group_lo >= group_hi) return MOE_ERR_SHAPE;
  if (T == 0) return MOE_OK;
  const int ns = moe_fused_shared_sets(T, H, E, K, I, Is);
  if (ns == 0) return MOE_ERR_SHAPE;
  if (!x || !src_of_row || !expert_offsets || !Wg || !Wu || !Wd || !Wsg || !Wsu || !Wsd || !Yp || !S_parts || !workspace)
    return MOE_ERR_NULL;
  if (wgate && !sg) return MOE_ERR_NULL;
  const int P = T * K;
  const int rows = P + ns * T;
  if (workspace_bytes < (size_t)rows * (size_t)I * 2) return MOE_ERR_WORKSPACE;   // h of the routed rows, then of every shared set
  const int mean_rows = (P + E - 1) / E;
  const Plan plan = make_plan(mean_rows, E, policy);
  if (!plan.valid || (policy & 0xff) == 9 || plan.tile_rows == 64) return MOE_ERR_SHAPE;
  GemmArgs gu{};
  gu.A = (const bf16_t*)x; gu.B0 = (const bf16_t*)Wg; gu.B1 = (const bf16_t*)Wu; gu.C = (bf16_t*)workspace;
  gu.offsets = expert_offsets; gu.lo = group_lo; gu.hi = group_hi; gu.ids = nullptr; gu.rows_total = rows;
  gu.mean_rows = mean_rows; gu.experts_layer = E; gu.N = I; gu.Kdim = H;
  gu.n_shared = ns; gu.shared_rows = T; gu.rows_routed = P;
  GemmArgs dn = gu;
  gu.gather = src_of_row; gu.gather_div = K;
  gu.Bs0 = (const bf16_t*)Wsg; gu.Bs1 = (const bf16_t*)Wsu; gu.shared_b_step = (long)I * H; gu.ldb_shared = H;
  gu.As = (const bf16_t*)x;                 // set s of the shared expert reads the tokens in order
  dn.A = (const bf16_t*)workspace; dn.B0 = (const bf16_t*)Wd; dn.B1 = nullptr; dn.C = (bf16_t*)Yp;
  dn.N = H; dn.Kdim = I;
  dn.Bs0 = (const bf16_t*)Wsd; dn.shared_b_step = I; dn.ldb_shared = Is;   // set s: columns [s*I, (s+1)*I) of Wsd [H,Is]
  dn.Cs = (bf16_t*)S_parts;
  int rc = 0, parts;
  const bool narrow = stream_narrow(mean_rows, H);     // (of gate/up; the down projection must be served alike)
  if (plan.stream && narrow == stream_narrow(mean_rows, I) && T <= (narrow ? FUSED_NARROW_T : FUSED_WIDE_T)) {
    // few rows per routed expert: the streaming kernels, whose launches take the shared sets along (the hidden rows of the
    // sets lie behind the routed ones: as one [T,Is] for the narrow kernel, as a [T,I] per set for the wide one)
    gu.rows_total = dn.rows_total = P;
    gu.Cs = (bf16_t*)workspace + (size_t)P * I;
    dn.As = gu.Cs;
    set_shared_parts(dn, ns, Is);
    if (narrow) gu.ldb_shared = Is;
    rc = ffn_forward(gu, dn, plan, (hipStream_t)stream, &parts);
  } else if (plan.stream) {
    // the routed rows go through the streaming kernels all the same (the bits of the plain block call), the shared sets,
    // with more tokens than passes over their weights pay for, through tiles of their own
    Plan tiles = plan;
    tiles.stream = false;
    GemmArgs sgu = gu, sdn = dn;
    sgu.offsets = sdn.offsets = nullptr; sgu.gather = nullptr; sgu.lo = sgu.hi = sdn.lo = sdn.hi = 0;
    sgu.rows_total = sdn.rows_total = ns * T;
    gu.n_shared = dn.n_shared = 0;
    gu.rows_total = dn.rows_total = P;
    rc = ffn_forward(gu, dn, plan, (hipStream_t)stream, &parts);
    if (rc == 0) rc = ffn_forward(sgu, sdn, tiles, (hipStream_t)stream, &parts);
  } else {
    rc = ffn_forward(gu, dn, plan, (hipStream_t)stream, &parts);
  }
  if (rc != 0) return rc;
  if (wgate && plan.do_down) return launch_gate_dot(x, wgate, T, H, sg, (hipStream_t)stream);
  return MOE_OK;
}

int moe_expert_group_forward(int group_lo, int group_hi, const void* Xp, const int32_t* expert_offsets,
                             const void* Wg, const void* Wu, const void* Wd, int P, int H, int E, int I, void* Yp,
                             void* workspace, size_t workspace_bytes, void* stream) {
  return moe_expert_group_forward_ex(group_lo, group_hi, Xp, expert_offsets, Wg, Wu, Wd, P, H, E, I, Yp, workspace,
                                     workspace_bytes, 0, stream);
}

}  // extern "C"

// gate_formed (nullptr: here): set to whether sg was formed; the caller then forms it where it was not
static int shared_forward_impl(const void* x, const void* Wsg, const void* Wsu, const void* Wsd, const void* wgate, int T,
                               int H, int Is, void* S, float* sg, void* workspace, size_t workspace_bytes, int policy,
                               void* stream, bool* gate_formed) {
  if (T < 0 || !dims_ok(H) || !dims_ok(Is)) return MOE_ERR_SHAPE;
  if ((long long)T * (H > Is ? H : Is) >= (1ll << 31)) return MOE_ERR_SHAPE;
  if (T == 0) return MOE_OK;
  if (!x || !Wsg || !Wsu || !Wsd || !S || !workspace) return MOE_ERR_NULL;
  if (wgate && !sg) return MOE_ERR_NULL;
  if (workspace_bytes < (size_t)T * (size_t)Is * 2) return MOE_ERR_WORKSPACE;   // h, bf16 [T,Is]
  Plan plan = make_plan(T, 1, policy);
  if (!plan.valid) return MOE_ERR_SHAPE;
  const bool few = (policy & 0xff) == 0 && T <= SHARED_FEW_T;
  const size_t h_bytes = align256((size_t)T * (size_t)Is * 2);
  // K parts of the down projection: as many as the sizes call for.  The 128x64 shape asked for by the caller and batches up
  // to 512 tokens must bring room for them; otherwise parts without room are formed in turn, to the same bits.
  const size_t one_part = (size_t)T * (size_t)H * 4;
  int room = (int)std::min<size_t>(SHARED_KPARTS_MAX, workspace_bytes > h_bytes ? (workspace_bytes - h_bytes) / one_part : 0);
  int parts_max = 0;
  if (!plan.stream && (plan.tile_rows == 64 || plan.tile_rows == 0) && tile_down_ksplit(Is) > 1) {
    const bool must = plan.tile_rows == 64 || T <= SHARED_SMALL_T;
    parts_max = must ? tile_down_ksplit(Is) : shared_parts_room(T, H);
    if (must && room < parts_max) return MOE_ERR_WORKSPACE;
  }
  // (memory behind h that holds the tokens or the output is no room)
  const void* const behind = static_cast<const unsigned char*>(workspace) + h_bytes;
  if (!apart(S, one_part / 2, behind, room * one_part) || !apart(x, one_part / 2, behind, room * one_part)) room = 0;
  const int few_parts = few && room >= shared_few_parts(Is) ? shared_few_parts(Is) : 1;   // (1: formed in turn)
  const bool side_by_side = few ? few_parts > 1 : room > 1 && parts_max > 1;
  float* part = side_by_side ? reinterpret_cast<float*>(static_cast<unsigned char*>(workspace) + h_bytes) : nullptr;
  GemmArgs gu{};
  gu.A = (const bf16_t*)x; gu.B0 = (const bf16_t*)Wsg; gu.B1 = (const bf16_t*)Wsu; gu.C = (bf16_t*)workspace;
  gu.offsets = nullptr; gu.lo = 0; gu.hi = 1; gu.rows_fixed = T; gu.rows_total = T; gu.mean_rows = T;
  gu.N = Is; gu.Kdim = H;
  GemmArgs dn = gu;
  dn.A = (const bf16_t*)workspace; dn.B0 = (const bf16_t*)Wsd; dn.B1 = nullptr; dn.C = (bf16_t*)S;
  dn.N = H; dn.Kdim = Is; dn.Cpart = part; dn.parts_max = parts_max; dn.parts_room = room;
  gu.leave_room = (policy >> 10) & 1;
  if (few) {
    plan.stream = true;
    gu.n_shared = 1;
    dn.n_shared = few_parts;
    set_shared_parts(dn, shared_few_parts(Is), Is);
    gu.shared_rows = dn.shared_rows = T;
    gu.ldb_shared = dn.ldb_shared = Is;
    gu.As = gu.A; gu.Bs0 = gu.B0; gu.Bs1 = gu.B1; gu.Cs = gu.C;
    dn.As = dn.A; dn.Bs0 = dn.B0; dn.Cs = dn.C;
  }
  int parts;
  const int rc = ffn_forward(gu, dn, plan, (hipStream_t)stream, &parts);
  if (rc != 0) return rc;
  if (few && plan.do_down) parts = few_parts;
  if (parts > 1) {   // the gate logits beside the sum, unless they go where it still reads
    const bool beside = wgate && apart(sg, (size_t)T * 4, part, (size_t)parts * one_part);
    const int rc_sum = launch_sum_parts(part, parts, T, H, S, x, beside ? wgate : nullptr, sg, (hipStream_t)stream);
    if (rc_sum != 0 || beside || !wgate) return rc_sum;
    return launch_gate_dot(x, wgate, T, H, sg, (hipStream_t)stream);
  }
  if (gate_formed != nullptr) {
    *gate_formed = false;
    return MOE_OK;
  }
  if (wgate && plan.do_down) return launch_gate_dot(x, wgate, T, H, sg, (hipStream_t)stream);
  return MOE_OK;
}

extern "C" {

int moe_shared_forward_ex(const void* x, const void* Wsg, const void* Wsu, const void* Wsd, const void* wgate, int T,
                          int H, int Is, void* S, float* sg, void* workspace, size_t workspace_bytes, int policy,
                          void* stream) {
  return shared_forward_impl(x, Wsg, Wsu, Wsd, wgate, T, H, Is, S, sg, workspace, workspace_bytes, policy, stream, nullptr);
}

int moe_shared_forward(const void* x, const void* Wsg, const void* Wsu, const void* Wsd, const void* wgate, int T,
                       int H, int Is, void* S, float* sg, void* workspace, size_t workspace_bytes, void* stream) {
  return moe_shared_forward_ex(x, Wsg, Wsu, Wsd, wgate, T, H, Is, S, sg, workspace, workspace_bytes, 0, stream);
}

int moe_combine(const void* Yp, const int32_t* row_of_pair, const float* topk_w, const void* S, const float* sg,
                int T, int H, int K, void* out, void* stream) {
  if (T < 0 || !dims_ok(H) || K < 1 || K > 16) return MOE_ERR_SHAPE;
  if (T == 0) return MOE_OK;
  if (!Yp || !row_of_pair || !topk_w || !out) return MOE_ERR_NULL;
  if ((S == nullptr) != (sg == nullptr)) return MOE_ERR_NULL;
  return launch_combine(Yp, row_of_pair, topk_w, S, 1, sg, T, H, K, out, (hipStream_t)stream);
}

int moe_combine_parts(const void* Yp, const int32_t* row_of_pair, const float* topk_w, const void* S_parts, int n_parts,
                      const float* sg, int T, int H, int K, void* out, void* stream) {
  if (T < 0 || !dims_ok(H) || K < 1 || K > 16 || n_parts < 1 || n_parts > MOE_SHARED_SETS_MAX) return MOE_ERR_SHAPE;
  if (T == 0) return MOE_OK;
  if (!Yp || !row_of_pair || !topk_w || !out || !S_parts || !sg) return MOE_ERR_NULL;
  return launch_combine(Yp, row_of_pair, topk_w, S_parts, n_parts, sg, T, H, K, out, (hipStream_t)stream);
}

int moe_layer_shared_sets(int T, int H, int E, int K, int I, int Is) {
  if (T < 1 || T > SHARED_FEW_T || K < 1 || E < 2 || I <= 0 || Is <= 0 || !dims_ok(H) || !dims_ok(I) || !dims_ok(Is)) return 0;
  if (((long long)T * K + E - 1) / E > STREAM_FEW_ROWS) return 0;
  const int sets = (Is + I - 1) / I;
  return sets <= MOE_SHARED_SETS_MAX ? sets : 0;
}

int moe_layer_forward(const void* x, const void* Wr, const float* bias, const int32_t* seg_offsets, int n_seg, const void* Wg,
                      const void* Wu, const void* Wd, const void* Wsg, const void* Wsu, const void* Wsd, const void* wgate,
                      int T, int H, int E, int K, int I, int Is, int renorm, int group_lo, int group_hi, int policy,
                      int shared_policy, int32_t* topk_ids, float* topk_w, int32_t* expert_offsets, int32_t* src_of_row,
                      int32_t* row_of_pair, void* Xp, void* Yp, void* S, float* sg, void* out, void* permute_workspace,
                      size_t permute_workspace_bytes, void* workspace, size_t workspace_bytes, void* shared_workspace,
                      size_t shared_workspace_bytes, float next_eps, void* next, void* stream) {
  if (next != nullptr && (H > 8192 || !(next_eps >= 0.0f))) return MOE_ERR_SHAPE;
  int rc = seg_offsets != nullptr
               ? moe_route_segments(x, Wr, bias, seg_offsets, n_seg, T, H, E, K, renorm, topk_ids, topk_w, stream)
               : moe_route(x, Wr, bias, T, H, E, K, renorm, topk_ids, topk_w, stream);
  if (rc != MOE_OK) return rc;
  rc = permute_refusal(topk_ids, x, T, H, E, K, expert_offsets, src_of_row, row_of_pair, Xp, permute_workspace,
                       permute_workspace_bytes);
  if (rc != MOE_OK) return rc;
  const int P = T * K, sets = moe_layer_shared_sets(T, H, E, K, I, Is);
  const size_t h_bytes = sets > 0 ? align256((size_t)T * (size_t)Is * 2) : 0;
  const int parts = shared_few_parts(Is);
  const size_t part_bytes = (size_t)parts * (size_t)T * (size_t)H * 4;
  const bool copied = Xp != nullptr;
  // The steps run one after another, so a caller may hand the same memory to several of them (one buffer as every
  // workspace, an output in a workspace that no later step reads).  What is done in one launch instead must not overlap:
  // a riding shared expert writes its hidden rows and parts while the block's launches read and write theirs, and its
  // parts are read while the aggregation writes.
  const size_t x_bytes = (size_t)T * (size_t)H * 2, pairs = (size_t)P * 4;
  const void* const riding = shared_workspace;
  const size_t riding_bytes = h_bytes + part_bytes;
  const bool ride = sets > 0 && policy == 0 && shared_policy == 0 && Wsg && Wsu && Wsd && S && sg && shared_workspace &&
                    shared_workspace_bytes >= riding_bytes && apart(riding, riding_bytes, workspace, (size_t)P * (size_t)I * 2) &&
                    (!copied || apart(riding, riding_bytes, Xp, (size_t)P * (size_t)H * 2)) &&
                    apart(riding, riding_bytes, src_of_row, pairs) &&
                    apart(riding, riding_bytes, expert_offsets, ((size_t)E + 1) * 4) &&
                    apart(riding, riding_bytes, sg, (size_t)T * 4) && apart(riding, riding_bytes, S, x_bytes) &&
                    apart(riding, riding_bytes, x, x_bytes) && apart(riding, riding_bytes, out, x_bytes) &&
                    apart(riding, riding_bytes, next, next ? x_bytes : 0);
  // The sort inside the experts' first launch: that launch then reads the ids and x, and writes the sorted arrays, beside
  // the hidden rows (and those of a riding shared expert).
  const size_t h_routed = (size_t)P * (size_t)I * 2, offsets_bytes = ((size_t)E + 1) * 4;
  const auto beside_hidden = [&](const void* p, size_t n) {
    return apart(p, n, workspace, h_routed) && (!ride || apart(p, n, riding, riding_bytes));
  };
  const bool sort_here = T > 0 && policy == 0 && sort_in_gateup(P, H, E, I, group_hi - group_lo) && beside_hidden(topk_ids, pairs) && beside_hidden(x, x_bytes) &&
                         beside_hidden(expert_offsets, offsets_bytes) && beside_hidden(src_of_row, pairs) &&
                         beside_hidden(row_of_pair, pairs) && apart(topk_ids, pairs, expert_offsets, offsets_bytes) &&
                         apart(topk_ids, pairs, src_of_row, pairs) && apart(topk_ids, pairs, row_of_pair, pairs) &&
                         (!copied || (apart(Xp, (size_t)P * (size_t)H * 2, x, x_bytes) && beside_hidden(Xp, (size_t)P * (size_t)H * 2)));
  if (!sort_here) {
    rc = launch_permute(topk_ids, x, T, H, E, K, expert_offsets, src_of_row, row_of_pair, Xp, permute_workspace, (hipStream_t)stream);
    if (rc != 0) return rc;
  }
  const Sort sort{topk_ids, expert_offsets, src_of_row, row_of_pair, Xp};
  Riders riders{x, Wsg, Wsu, Wsd, shared_workspace, nullptr, sets, parts, T, Is};
  if (ride) riders.part = reinterpret_cast<float*>(static_cast<unsigned char*>(shared_workspace) + h_bytes);
  // The shared expert's hidden rows formed beside the routed ones: nothing that the routed experts still read or write may
  // lie there, and everything its own call would refuse is left to that call.
  const size_t shared_h = (size_t)T * (size_t)Is * 2;
  const bool host = !ride && T > 0 && Is > 0 && dims_ok(H) && dims_ok(I) && dims_ok(Is) && policy == 0 && shared_policy == 0 &&
                    Wsg && Wsu && Wsd && S && shared_workspace && shared_workspace_bytes >= shared_h && (!wgate || sg) &&
                    (Is + I - 1) / I <= MOE_SHARED_SETS_MAX && (long long)T * (H > Is ? H : Is) < (1ll << 31) &&
                    apart(shared_workspace, shared_h, workspace, h_routed) && apart(shared_workspace, shared_h, x, x_bytes) &&
                    apart(shared_workspace, shared_h, Yp, (size_t)P * (size_t)H * 2) && apart(workspace, h_routed, x, x_bytes) &&
                    apart(Yp, (size_t)P * (size_t)H * 2, x, x_bytes) &&
                    (!copied || apart(shared_workspace, shared_h, Xp, (size_t)P * (size_t)H * 2)) &&
                    apart(shared_workspace, shared_h, src_of_row, pairs) && apart(shared_workspace, shared_h, expert_offsets, offsets_bytes);
  const Hosted hosted{x, Wsg, Wsu, shared_workspace, T, Is};
  bool is_hosted = false;
  const bool from_x = sort_here || !copied;
  rc = expert_group_forward_impl(group_lo, group_hi, nullptr, from_x ? x : Xp, from_x ? src_of_row : nullptr, from_x ? K : 1,
                                 expert_offsets, Wg, Wu, Wd, P, H, E, I, Yp, workspace, workspace_bytes, policy, stream,
                                 ride ? &riders : nullptr, sort_here ? &sort : nullptr, host ? &hosted : nullptr, &is_hosted);
  if (sort_here && (rc == MOE_ERR_NULL || rc == MOE_ERR_SHAPE || rc == MOE_ERR_WORKSPACE)) {   // refused: the step before it stands
    const int rc_sort = launch_permute(topk_ids, x, T, H, E, K, expert_offsets, src_of_row, row_of_pair, Xp, permute_workspace, (hipStream_t)stream);
    if (rc_sort != 0) return rc_sort;
  }
  if (rc != MOE_OK) return rc;
  // The aggregation forms the gate logit and the residual step where no row that it still reads for another token lies
  // in what it writes for this one (x itself may be out or next: then the rows are the token's own); otherwise they are
  // launches of their own in their places.
  const bool x_kept = (out == x || apart(out, x_bytes, x, x_bytes)) && (!next || next == x || apart(next, x_bytes, x, x_bytes));
  const bool next_here = next != nullptr && x_kept && out != x && apart(next, x_bytes, Yp, (size_t)P * (size_t)H * 2) &&
                         apart(next, x_bytes, S, S ? x_bytes : 0) && apart(next, x_bytes, sg, sg ? (size_t)T * 4 : 0) &&
                         apart(next, x_bytes, row_of_pair, pairs) && apart(next, x_bytes, topk_w, pairs) &&
                         (next == out || apart(next, x_bytes, out, x_bytes));
  bool gate_formed = true;   // sg complete (or no shared expert)
  if (!ride && Is > 0) {
    rc = shared_forward_impl(x, Wsg, Wsu, Wsd, wgate, T, H, Is, S, sg, shared_workspace, shared_workspace_bytes,
                             is_hosted ? shared_policy | 0x200 : shared_policy, stream, T > 0 && x_kept && (shared_policy & 0x300) == 0 ? &gate_formed : nullptr);
    if (rc != MOE_OK) return rc;
  }
  if (T == 0) return MOE_OK;
  if (!out || (Is > 0 && (!S || !sg))) return MOE_ERR_NULL;
  if (ride && !x_kept && wgate) {
    rc = launch_gate_dot(x, wgate, T, H, sg, (hipStream_t)stream);
    if (rc != MOE_OK) return rc;
  }
  rc = launch_combine_layer(Yp, row_of_pair, topk_w, ride ? riders.part : nullptr, parts, x,
                            x_kept && (ride || !gate_formed) ? wgate : nullptr, Is > 0 ? S : nullptr, sg, T, H, K, out, next_eps,
                            next_here ? next : nullptr, (hipStream_t)stream);
  if (rc != MOE_OK || next == nullptr || next_here) return rc;
  return launch_residual_norm(x, out, T, H, next_eps, next, (hipStream_t)stream);
}

int moe_residual_norm(const void* x, const void* y, int T, int H, float eps, void* out, void* stream) {
  if (T < 0 || !dims_ok(H) || H > 8192 || !(eps >= 0.0f)) return MOE_ERR_SHAPE;
  if (T == 0) return MOE_OK;
  if (!x || !y || !out) return MOE_ERR_NULL;
  return launch_residual_norm(x, y, T, H, eps, out, (hipStream_t)stream);
}

}  // extern "C"
