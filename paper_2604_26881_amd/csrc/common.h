// Shared device helpers for the gfx950 MoE-layer kernels (wave64, CDNA4).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>
#include <atomic>

namespace moe {

typedef uint16_t bf16_t;  // raw bf16 bits
typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(16))) float f32x16;
typedef __attribute__((ext_vector_type(4))) float f32x4;
typedef __attribute__((ext_vector_type(4))) uint32_t u32x4;   // 16 bytes moved as one register quad

constexpr int WAVE = 64;

__device__ __forceinline__ float bf16_lo(uint32_t packed) { return __uint_as_float(packed << 16); }
__device__ __forceinline__ float bf16_hi(uint32_t packed) { return __uint_as_float(packed & 0xffff0000u); }

// fp32 -> bf16, round to nearest even (finite inputs).
__device__ __forceinline__ uint32_t f32_to_bf16_bits(float f) {
  uint32_t u = __float_as_uint(f);
  u += 0x7fffu + ((u >> 16) & 1u);
  return u >> 16;
}
// Two fp32 -> packed bf16 pair, round to nearest even: one v_cvt_pk_bf16_f32 on gfx950 (the same
// result as f32_to_bf16_bits for finite values).
typedef __attribute__((ext_vector_type(2))) float f32x2;
typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2;
__device__ __forceinline__ uint32_t pack_bf16x2(float lo, float hi) {
  const f32x2 v = {lo, hi};
  return __builtin_bit_cast(uint32_t, __builtin_convertvector(v, bf16x2));
}

__device__ __forceinline__ bf16x8 as_bf16x8(u32x4 v) { return __builtin_bit_cast(bf16x8, v); }

__device__ __forceinline__ float wave_sum(float v) {
#pragma unroll
  for (int s = 32; s >= 1; s >>= 1) v += __shfl_xor(v, s, WAVE);
  return v;
}
__device__ __forceinline__ float wave_max(float v) {
#pragma unroll
  for (int s = 32; s >= 1; s >>= 1) v = fmaxf(v, __shfl_xor(v, s, WAVE));
  return v;
}

// Lanes l < 32 and l + 32 trade registers: afterwards a holds, in lanes 32-63, what b held in lanes
// 0-31, and b holds, in lanes 0-31, what a held in lanes 32-63 (v_permlane32_swap); the other
// halves keep their values.
__device__ __forceinline__ void trade_halves(uint32_t& a, uint32_t& b) {
  const auto r = __builtin_amdgcn_permlane32_swap(a, b, false, false);
  a = r[0];
  b = r[1];
}

// One 16-byte-per-lane copy from global memory straight into LDS (no registers in between):
// lane l of the wave writes LDS bytes [lds + 16*l, +16) from global address base + voff.
// The copy is asynchronous; it is counted by vmcnt like any other vector memory load.
// (One wait state between the write of m0 and the instruction that reads it: the ISA asks for it, and the
// compiler, which pads its own such pairs, does not look inside an asm statement.)
// once (a constant after inlining): the non-temporal hint, for data that is read once (streamed weights), so that it does not
// displace reusable lines from the caches.  Measured on a 1 GiB stream of 4 KB rows: 6.0 TB/s without
// the hint, 6.8 TB/s with it.
__device__ __forceinline__ void copy_to_lds_16(const void* base, uint32_t voff, uint32_t lds, bool once = false) {
  if (once)
    asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1 nt" ::"v"(voff), "s"(base), "s"(lds)
                 : "memory", "m0");
  else
    asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1" ::"v"(voff), "s"(base), "s"(lds)
                 : "memory", "m0");
}
template <int N>
__device__ __forceinline__ void wait_copies_but() {   // all but the N most recent copies have landed
  asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory");
}
__device__ __forceinline__ void workgroup_barrier() { asm volatile("s_barrier" ::: "memory"); }
__device__ __forceinline__ void wait_lds_reads() { asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory"); }

// Launch helpers used by the C entry points.
struct GemmArgs {
  const bf16_t* A;     // token rows [rows, Kdim]
  const bf16_t* B0;    // weights [E, N, Kdim]  (gate branch, or the down projection)
  const bf16_t* B1;    // weights of the up branch (gate/up kernels), else unused
  bf16_t* C;           // output rows [rows, N]
  const int32_t* offsets;  // expert_offsets on the device, or nullptr for one expert on rows [0, rows_fixed)
  int lo, hi;          // experts [lo, hi); with an id list: positions [lo, hi) of the list
  const int32_t* ids;  // nullptr: expert id = position; else the block is the experts ids[lo .. hi) (device memory)
  int rows_fixed;
  int rows_total;      // number of rows of A and C (upper bound used to size the grid)
  int mean_rows;       // expected rows per expert (rows_total / experts of the layer): picks kernel shapes
  int experts_layer;   // routed experts of the layer (0: one weight set): with mean_rows, the tiles of the whole layer
  int N;               // output columns (per branch for gate/up)
  int Kdim;            // contraction length
  float* Cpart;        // room for the fp32 partial outputs [parts, rows_total, N] of kernels that cut K, else unused
  int parts_max;       // most parts the sizes call for (0 and 1: no cut); the number, and with it the result, does not depend
                       // on the parts that Cpart has room for (parts_room)
  const int32_t* gather;   // nullptr: row r of A is A[r]; else row r of A is A[gather[r] / gather_div]
  int gather_div;          // (the token rows themselves, addressed through src_of_row: no permuted copy)
  int leave_room;          // 1: small kernels run on other streams meanwhile: no tile shape that holds them up for long
                           // (pick_tile_shape says which)
  // Shared experts riding along with a routed block (tile kernels; n_shared == 0: none; the kernel that streams the weights
  // of a few rows takes them too, as its comment states).  They are
  // n_shared more weight sets, each applied to all shared_rows tokens.  In the row space of A and C
  // the routed rows are [0, rows_routed) and set s owns rows rows_routed + s*shared_rows onwards.
  int n_shared;
  int shared_rows;         // tokens T
  int rows_routed;         // P
  const bf16_t* Bs0;       // weights of set 0 (gate branch, or the down projection); set s starts s*shared_b_step
  const bf16_t* Bs1;       // elements further on; consecutive weight rows of a set are ldb_shared elements apart
  long shared_b_step;
  int ldb_shared;
  const bf16_t* As;        // not nullptr: set s reads its token rows from As[0 .. shared_rows) instead of A (gate/up: x)
  bf16_t* Cs;              // not nullptr: row r of set s goes to Cs[s*shared_rows + r] instead of C (down: the S parts)
  int shared_cols;         // (tile kernels, gate/up) not 0: set s is columns [s*N, (s+1)*N) of one hidden layer of this many, in
                           // Cs [shared_rows, shared_cols] (the last set may be narrower)
  // Measurement aid (tile kernels; nullptr: off): workgroup b < clock_groups writes four values at clocks[4*b]:
  // shader-clock ticks and ticks of the constant 100 MHz clock between its start and its end, the shader-clock
  // ticks it spent inside the K loops of its tiles, and the number of its tiles.
  long long* clocks;
  int clock_groups;
  int parts_room;          // parts that Cpart has room for; more of them are formed in turn
  int shared_parts;        // (streaming kernel, down) K parts of the shared contraction, of part_steps steps of 64 each,
  int part_steps;          // the first part_extra of them one more
  int part_extra;
  // (narrow streaming kernel, gate/up of a few pairs) not nullptr: the micro-batch is constructed in this launch, from these
  // expert ids of the n_pairs = T * K pairs; offsets and gather are written by it, and read by later launches only
  const int32_t* sort_ids;
  int n_pairs;
  int32_t* sort_offsets;   // [experts_layer + 1]
  int32_t* sort_src;       // src_of_row
  int32_t* sort_rows;      // row_of_pair
  bf16_t* sort_copy;       // not nullptr: the permuted copy Xp of the token rows (A)
  int rot_shift;           // (tile kernels) log2 of the output columns that share a K start: those of a tile of the layer's shape
};
// Raises a kernel's dynamic LDS limit once per device: one bit per device id in `done` (the kernel's own),
// set after the call has succeeded there (two threads may both make the call; it is idempotent).
inline int raise_lds_limit(const void* kern, int lds, std::atomic<uint64_t>& done) {
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess) return -4;
  const uint64_t bit = 1ull << (dev & 63);
  if (dev >= 64 || !(done.load(std::memory_order_acquire) & bit)) {
    if (hipFuncSetAttribute(kern, hipFuncAttributeMaxDynamicSharedMemorySize, lds) != hipSuccess) return -4;
    if (dev < 64) done.fetch_or(bit, std::memory_order_release);
  }
  return 0;
}

// Where the tile-kernel launches of the calling host thread record their clocks (nullptr: nowhere).
void set_tile_clock_buffer(long long* clocks, int groups);

// bias [E] for all tokens (seg == nullptr), or bias [n_seg, E] with seg [n_seg + 1] segment bounds on the device
int launch_route(const void* x, const void* Wr, const float* bias, const int32_t* seg, int n_seg, int T, int H, int E,
                 int K, int renorm, int32_t* ids, float* w, hipStream_t st);
// Lanes of the wave whose (valid) pair has the same expert id as this lane's
__device__ __forceinline__ unsigned long long match_expert(int e, bool valid, int nbits) {
  unsigned long long match = __ballot(valid);
  for (int b = 0; b < nbits; ++b) {
    const unsigned long long bal = __ballot(valid && ((e >> b) & 1));
    match &= ((e >> b) & 1) ? bal : ~bal;
  }
  return match;
}
__device__ __forceinline__ int bits_for(int E) {
  int nbits = 0;
  while ((1 << nbits) < E) ++nbits;
  return nbits;
}
int launch_permute(const int32_t* ids, const void* x, int T, int H, int E, int K, int32_t* offsets,
                   int32_t* src_of_row, int32_t* row_of_pair, void* Xp, void* workspace, hipStream_t st);
int launch_combine(const void* Yp, const int32_t* row_of_pair, const float* w, const void* S, int n_parts,
                   const float* sg, int T, int H, int K, void* out, hipStream_t st);
// The aggregation of a layer with what else it can do on the way: with part (not nullptr) S = the `parts` fp32 tensors
// [T,H] added in ascending part; with wgate sg = <x, wgate>; with next also next = residual_norm(x, out), H <= 8192.
int launch_combine_layer(const void* Yp, const int32_t* row_of_pair, const float* w, const float* part, int parts,
                         const void* x, const void* wgate, void* S, float* sg, int T, int H, int K, void* out, float eps,
                         void* next, hipStream_t st);
int launch_residual_norm(const void* x, const void* y, int T, int H, float eps, void* out, hipStream_t st);
// C = the `parts` fp32 tensors [T,H] of a K-cut down projection, added in ascending part; with wgate also sg = <x, wgate>
int launch_sum_parts(const float* part, int parts, int T, int H, void* C, const void* x, const void* wgate, float* sg,
                     hipStream_t st);
int launch_gate_dot(const void* x, const void* wgate, int T, int H, float* sg, hipStream_t st);
int launch_mfma_probe(const void* operands, int iters, int workgroups, long long* clocks, hipStream_t st);
// Tiled MFMA kernels (many rows per expert) and streaming kernels (few rows per expert).
int launch_tile_gateup(const GemmArgs& a, int tile_rows, hipStream_t st);
int launch_tile_down(const GemmArgs& a, int tile_rows, hipStream_t st, int* parts);
// Whether the gate/up launch of a layer takes the shared expert's gate/up tiles along (a: the routed experts' arguments)
bool tile_hosts_shared(const GemmArgs& a, int tokens, int Is);
int tile_down_ksplit(int Kdim);   // most K parts of the down projection
constexpr int STREAM_FEW_ROWS = 6;   // mean rows per expert up to which the narrow one of them serves a layer
// It also serves contractions of up to four K steps, where what counts is how soon a wave starts: 16 experts of H 256, I 256
// at 7 to 26 rows, gate/up + down: 7.4-8.7 us narrow, 9.1-11 wide.
inline bool stream_narrow(int mean_rows, int Kdim) { return mean_rows <= STREAM_FEW_ROWS || Kdim <= 256; }
constexpr int SORT_HERE_MAX = 128;   // most pairs whose micro-batch that kernel's gate/up launch constructs as well (sort_in_gateup draws the line)
// Streaming kernels that stage the weights through wave-private LDS rings (whole-line requests): a few rows per
// expert, and up to a few dozen.
int launch_stream_lds_gateup(const GemmArgs& a, hipStream_t st);
int launch_stream_lds_down(const GemmArgs& a, hipStream_t st);
int launch_stream_wide_gateup(const GemmArgs& a, hipStream_t st);
int launch_stream_wide_down(const GemmArgs& a, hipStream_t st);

}  // namespace moe
