// Order-preserving gather-compaction of the cache rows (App. B: K' = K[keep_idx], V' = V[keep_idx]).
//
// In place, destination row j and source row keep_idx[j] live in the same buffer.  keep_idx is strictly
// ascending, so keep_idx[j] >= j: a row only ever moves towards the front.  One workgroup walks the destination
// rows of one (unit, tensor) in ascending chunks; inside a chunk every source row is first loaded into registers,
// then the workgroup synchronises, then the rows are stored.  A store of chunk c lands in rows
// [c*R, (c+1)*R), and every later chunk reads only rows >= (c+1)*R, so the only reads a store could overtake
// are those of its own chunk, which the barrier orders.  A tensor that is
// moved out of place beside one in place takes the same code without the barrier; both out of place: gather_rows_kernel.
#include <algorithm>

#include "ccd_common.h"
#include "ccd_rope.h"
#include "ccd_select_body.h"
#include "ccd_ticket.h"

namespace ccd {

namespace {

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

// Non-temporal 16-byte store: the compacted rows are not read again by this call, and marking them as streaming
// keeps them from lingering as dirty lines that the next kernel's reads would have to push out (measured: 9 us
// less for the compaction itself, 3 us less for the score pass that follows; streaming loads save another 3 us).
__device__ __forceinline__ void store_streaming(char* p, const uint4& v) {
  const u32x4 t = {v.x, v.y, v.z, v.w};
  __builtin_nontemporal_store(t, reinterpret_cast<u32x4*>(p));
}
// the source rows are read once as well
__device__ __forceinline__ uint4 load_streaming(const char* p) {
  const u32x4 t = __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(p));
  return make_uint4(t.x, t.y, t.z, t.w);
}

constexpr int kCpThreads = 1024;          // compaction of a kept list that is ready in memory
constexpr int kCpUnroll = 4;

// Appending a chunk of new context behind the cached tokens (Sec. 3.2: the pot is filled until it is full): rows
// [n, n + count) of every unit of K and V take the chunk's rows, dense [units, count, d] on the source side.  A unit's
// share is one contiguous run on both sides; the grid is (tensor, unit, segment of 16 KiB), 16 bytes per lane and
// four loads in flight (a store waits for all of them, and for the store before it).  Bound by HBM (256 units, 2048 tokens: 537 MB
// in 84 us) or, for a few units, by how many compute
// units take part: segments of 64 KiB gave 85 us, and 8.8 instead of 5.4 us for 8 units of 2048 tokens.  (Where chunk and pot stay in
// the memory-side cache from one call to the next, 130 to 270 MB in all, those of 64 KiB were 4 to 11 % faster.)
// values_first: the values of all units and then the keys, when chunk and pot together are more than the memory-side cache holds: the score
// pass that comes next reads the keys, and finds twice as many of them there as with keys and values in turn (append + distill, 256 units of
// 4096 tokens: given normalisers 337 -> 329 us, window and CaP keys 404 -> 389 us; 640 units 922 -> 911 us; 48 units of 13504 tokens 256 -> 239 us).
// Where it holds all of them, keys last is slower: they are what is left to write back when the kernel ends (33 units of 1376 tokens 37.2 ->
// 37.8 us, 8 of 7232 tokens 57.4 -> 58.1 us).
// stretch: a chunk that fills an empty pot is one stretch of memory on both sides, and cut into segments as a whole.  With segments of its own for
// every unit, whose last one is not full, the workgroups fall out of step with the 16 KiB that follow each other in memory, which costs
// more in one walk over the values than in turn: 208 units of 13710 tokens (214.2 segments each), in turn / values first / in one stretch
// 529 / 586 / 496 us, with their distillation 1083 / 1120 / 1043; 400 of 4144 (64.75) 319 / 336 / 294 and 660 / 668 / 630; 72 of 18528 (289.5) 255 /
// 246 / 235 and 554 / 525 / 515; 208 of 13696 (214) 516 / 504 / 504 and 1075 / 1061 / 1060.  (Into a pot that holds tokens already, values
// first: 14 sizes 0.997 to 1.038 times faster, whatever the last segment.)
// Append + distill of 128 to 640 units of 1536 to 9001 tokens, with and without CR-RoPE (whose scores read other keys), in one stretch against
// in turn: 1.02 to 1.085 times faster above 1 GB; up to there 1.00 to 1.04, but for six calls of 568 MB and 1 GB (0.977 to 0.998), whose compaction
// finds less in the cache.
// Carried novelty follows: entry n + j of every head takes the chunk's novelty of token j, kApNovelty tokens to a workgroup that also moves
// keys (one workgroup per head, one entry per thread after the other: 32768 tokens of 8 units 57 instead of 37 us).  In a stretch every
// nov_spread-th key workgroup takes the next kApNovelty tokens of the rows of novelty.
constexpr int kApThreads = 256;
constexpr int kApLoads = 4;
constexpr int kApNovelty = 1024;       // a multiple of the tokens of a segment (32, 64 or 128)
constexpr int64_t kMemorySideCache = 256 << 20;
constexpr int kApSegBytes = kApThreads * 16 * kApLoads;     // bytes one workgroup moves: 16 KiB
template <bool STRETCH>
__global__ __launch_bounds__(kApThreads) void append_rows_kernel(Dims D, int esz, int count, int segs, char* K, char* V,
                                                                 const char* Knew, const char* Vnew, float* novelty,
                                                                 const float* nov_new, int nov_per_head, int values_first, int nov_spread) {
  const int units = STRETCH ? 1 : D.units_run;   // (all units are one: segs of the whole stretch, offsets of unit 0)
  const int seg = blockIdx.x % segs;
  const int ut = blockIdx.x / segs;
  const bool isV = values_first ? ut < units : ut & 1;
  const int unit = D.unit0 + (values_first ? (isV ? ut : ut - units) : ut >> 1);
  const UnitIdx ui = decode_unit(D, unit);
  const int64_t run = (int64_t)count * D.d * esz * (STRETCH ? D.units : 1);      // bytes of a unit's share
  char* dst = (isV ? V : K) + (kv_offset(D, ui) + (int64_t)D.n * D.d) * esz;
  const char* src = (isV ? Vnew : Knew) + (int64_t)unit * run;
  const int64_t b0 = (int64_t)seg * kApSegBytes + threadIdx.x * 16;
  uint4 v[kApLoads];
#pragma unroll
  for (int i = 0; i < kApLoads; ++i) {
    const int64_t b = b0 + i * (kApThreads * 16);
    if (b < run) v[i] = load_streaming(src + b);
  }
  // (one key workgroup in 8 to 32: those whose segment starts at a multiple of kApNovelty tokens)
  int t_seg = seg * (kApSegBytes / (D.d * esz));
  UnitIdx un = ui;
  bool carry = novelty != nullptr && !isV;
  if (!STRETCH) {
    carry = carry && t_seg % kApNovelty == 0 && (nov_per_head || (ui.l == 0 && ui.h == 0));
  } else if (carry) {
    const int per_row = (count + kApNovelty - 1) / kApNovelty, piece = seg / nov_spread, row = piece / per_row;
    carry = seg % nov_spread == 0 && row < (nov_per_head ? D.units : D.B);
    t_seg = (piece - row * per_row) * kApNovelty;
    un = decode_unit(D, nov_per_head ? row : row * (D.L * D.Hkv));
  }
  if (carry) {
    const float* ns = nov_new + (int64_t)un.b * count;
    float* nd = novelty + nov_offset(D, un) + D.n;
    float nv[kApNovelty / kApThreads];
#pragma unroll
    for (int i = 0; i < kApNovelty / kApThreads; ++i) nv[i] = ns[min(t_seg + i * kApThreads + (int)threadIdx.x, count - 1)];
#pragma unroll
    for (int i = 0; i < kApNovelty / kApThreads; ++i) {
      const int j = t_seg + i * kApThreads + (int)threadIdx.x;
      if (j < count) nd[j] = nv[i];
    }
  }
#pragma unroll
  for (int i = 0; i < kApLoads; ++i) {
    const int64_t b = b0 + i * (kApThreads * 16);
    if (b < run) {          // the keys are read again by the next score pass, the values not before the compaction
      if (isV) store_streaming(dst + b, v[i]);
      else     *reinterpret_cast<uint4*>(dst + b) = v[i];
    }
  }
}

// All loads have arrived.  The builtin, so that the compiler knows it too: behind inline assembly it took the registers of loads
// under a condition for still in use and waited before every load and every store of the next rows.  Append + distill: 64 units of 2500 /
// 20000 tokens 77.7 / 497.6 -> 76.6 / 489.8 us, 128 units of 3000 tokens 142.5 -> 139.1 us; with that four rows per thread where one
// workgroup has a unit, not two: 256 units of 600 tokens 64.0 -> 62.9 us, 640 units of 2000 tokens 506.7 -> 502.1 us.
__device__ __forceinline__ void wait_for_loads() {
  asm volatile("" ::: "memory");
  __builtin_amdgcn_s_waitcnt(0x0F70);          // vmcnt(0); expcnt and lgkmcnt as they are
  asm volatile("" ::: "memory");
}

// Indices that have arrived before anything is loaded by them under a condition: where the compiler cannot count the loads in flight,
// the wait for the next index is one for the rows before it.
template <int N>
__device__ __forceinline__ void arrived(int (&v)[N]) {
#pragma unroll
  for (int i = 0; i < N; ++i) asm volatile("" : "+v"(v[i]));
}

template <int ROWB>
__global__ __launch_bounds__(kCpThreads) void compact_rows_kernel(Dims D, const char* Ksrc, const char* Vsrc,
                                                                  const int32_t* __restrict__ keep_idx, char* Kdst,
                                                                  char* Vdst) {
  constexpr int kLanesPerRow = ROWB / 16;
  constexpr int kRowsPerPass = kCpThreads / kLanesPerRow;
  const int unit = D.unit0 + (blockIdx.x >> 1);
  const bool isV = blockIdx.x & 1;
  const int64_t ubytes = kv_offset(D, decode_unit(D, unit)) * (int64_t)(ROWB / D.d);
  const char* src = (isV ? Vsrc : Ksrc) + ubytes;
  char* dst = (isV ? Vdst : Kdst) + ubytes;
  const bool inplace = (src == dst);
  const int32_t* keep = keep_idx + (int64_t)unit * D.k;
  const int lane_off = (threadIdx.x % kLanesPerRow) * 16;
  const int row_in_pass = threadIdx.x / kLanesPerRow;

  for (int base = 0; base < D.k; base += kRowsPerPass * kCpUnroll) {
    uint4 v[kCpUnroll];
    bool move[kCpUnroll];
    int sidx[kCpUnroll];
#pragma unroll
    for (int i = 0; i < kCpUnroll; ++i) sidx[i] = keep[min(base + i * kRowsPerPass + row_in_pass, D.k - 1)];
    arrived(sidx);
#pragma unroll
    for (int i = 0; i < kCpUnroll; ++i) {
      const int j = base + i * kRowsPerPass + row_in_pass;
      sidx[i] = min(max(sidx[i], 0), D.n_cap - 1);   // a corrupt index must not leave the pot
      move[i] = j < D.k && !(inplace && sidx[i] == j);
      if (move[i]) v[i] = load_streaming(src + (int64_t)sidx[i] * ROWB + lane_off);
    }
    wait_for_loads();
    if (inplace) __syncthreads();
#pragma unroll
    for (int i = 0; i < kCpUnroll; ++i) {
      const int j = base + i * kRowsPerPass + row_in_pass;
      if (move[i]) store_streaming(dst + (int64_t)j * ROWB + lane_off, v[i]);
    }
  }
}

// Out of place nothing orders the rows: (unit, tensor, run of destination rows) per workgroup, four rows per lane, three of them in
// flight (the compiler puts the first row's load behind the test that guards its store).
// Bound by HBM; the kernel above has two workgroups per unit, which leave the chip idle with few units (45 units, 3001 -> 1499
// rows of 128 bytes: 17.4 -> 8.3 us).
constexpr int kGaThreads = 256;
constexpr int kGaRows = 4;
template <int ROWB>
__global__ __launch_bounds__(kGaThreads) void gather_rows_kernel(Dims D, int segs, const char* __restrict__ Ksrc,
                                                                 const char* __restrict__ Vsrc,
                                                                 const int32_t* __restrict__ keep_idx, char* __restrict__ Kdst,
                                                                 char* __restrict__ Vdst) {
  constexpr int kLanesPerRow = ROWB / 16;
  constexpr int kRowsPerPass = kGaThreads / kLanesPerRow;
  const int seg = blockIdx.x % segs, ut = blockIdx.x / segs;
  const int unit = D.unit0 + (ut >> 1);
  const bool isV = ut & 1;
  const int64_t ubytes = kv_offset(D, decode_unit(D, unit)) * (int64_t)(ROWB / D.d);
  const char* src = (isV ? Vsrc : Ksrc) + ubytes;
  char* dst = (isV ? Vdst : Kdst) + ubytes;
  const int32_t* keep = keep_idx + (int64_t)unit * D.k;
  const int lane_off = (threadIdx.x % kLanesPerRow) * 16;
  const int j0 = seg * (kRowsPerPass * kGaRows) + threadIdx.x / kLanesPerRow;
  int sidx[kGaRows];
#pragma unroll
  for (int i = 0; i < kGaRows; ++i) sidx[i] = keep[min(j0 + i * kRowsPerPass, D.k - 1)];
  uint4 v[kGaRows];
#pragma unroll
  for (int i = 0; i < kGaRows; ++i)      // (a corrupt index must not leave the pot)
    v[i] = load_streaming(src + (int64_t)min(max(sidx[i], 0), D.n_cap - 1) * ROWB + lane_off);
#pragma unroll
  for (int i = 0; i < kGaRows; ++i) {
    const int j = j0 + i * kRowsPerPass;
    if (j < D.k) store_streaming(dst + (int64_t)j * ROWB + lane_off, v[i]);
  }
}

// per-head novelty carried with the cache: nov[j] <- nov[keep_idx[j]], same chunk discipline
__global__ __launch_bounds__(kCpThreads) void compact_novelty_kernel(Dims D, const int32_t* __restrict__ keep_idx,
                                                                     float* novelty) {
  const int unit = D.unit0 + blockIdx.x;
  float* nov = novelty + nov_offset(D, decode_unit(D, unit));
  const int32_t* keep = keep_idx + (int64_t)unit * D.k;
  for (int base = 0; base < D.k; base += kCpThreads) {
    const int j = base + threadIdx.x;
    float v = 0.f;
    if (j < D.k) v = nov[min(max(keep[j], 0), D.n_cap - 1)];
    wait_for_loads();
    __syncthreads();
    if (j < D.k) nov[j] = v;
  }
}

// Selection and compaction of a unit in one kernel (ccd_compress, rows of up to 32768 tokens): the kept list stays in LDS
// and K and V rows move together.  Against a selection kernel followed by a compaction kernel this saves a launch, the drain
// of a latency-bound grid, and the trip of keep_idx through memory.
//
// One workgroup per unit when the units fill the chip: it walks the destination rows in ascending chunks (see the top of
// the file) and is bound by HBM (80 us for 537 MB: 6.7 TB/s), behind about 10 us of selection.
//
// SHARED (few units): several workgroups per unit.  Each runs the whole selection for itself - same inputs, same list -
// and then draws chunks of the unit's destination rows by ticket.  A chunk's sources are loaded into registers and the
// chunk is marked as loaded; it is stored once all chunks BEFORE it are marked, since those are the only ones whose sources
// (keep[j] >= j) it can overwrite.  A workgroup draws tickets while it runs, and between a draw and its mark it waits at
// most for smaller chunks: the owner of the smallest unmarked chunk therefore never waits, and no order of dispatch and no
// number of resident workgroups can make anybody wait for ever.  Nothing has to be made visible but the marks
// themselves: a chunk's loads are complete before its mark, and nobody reads rows that were stored.
// Against dealing out column segments to at most eight workgroups per unit: 8 units, 2048 -> 1024, 23 -> 13 us with the
// carried novelty, which took a kernel of its own; 8 units, 32768 -> 4096: 113 -> 57 us.
//
// Threads: the moving of one workgroup per unit wants 16 waves (512 threads with twice the rows each: 2 - 3 us slower on 256
// units), a selection on a unit's share of the chip is faster with eight (tiny and single-layer calls: 1 - 2 us) as long as the row
// gives a thread little to do.  SHARED, append + distill with eight against 16 waves: 8 units of 3000 / 4096 tokens 38.2 / 40.5 against 37.6 /
// 40.9 us, of 4500 / 6000 / 8192 tokens 51.6 / 56.2 / 61.9 against 50.5 / 53.5 / 59.3; 64 of 8000 196 against 194; rows held in LDS 203 against 191.  (16 waves, 9000 / 16384 tokens in LDS against registers: 70.8 / 91.3
// against 68.9 / 89.1 us; one workgroup per unit the same.)
constexpr int kFewWavesTokens = 4096;
constexpr int sc_threads(bool shared, int n) { return shared && n <= kFewWavesTokens ? 512 : 1024; }      // (at most two chunks of tokens per thread)
// Waves per SIMD to compile for: 64 registers instead of 72 for rows of up to 4096 tokens, so that two workgroups fit a compute unit
// when there are more units than these: one selects while the other one moves rows, and the last round is not alone (append +
// distill with given normalisers, 2000 tokens: 400 / 640 units 257 / 438 -> 251 / 427 us, 600 tokens 85 / 129 -> 78 / 121 us; up to 256
// units the same; 300 units of 2000 tokens 182 -> 186 us).  With CR-RoPE 13 registers would be spilled (256 units 363 -> 383 us).
constexpr int sc_min_waves(bool shared, int chunks, int rope_row) { return !shared && chunks == 1 && rope_row == 0 ? 8 : 1; }
// Rows per thread and chunk.  ROPE: its coefficients take as many registers again, and four rows spilled 4 of them.
constexpr int sc_unroll(bool rope) { return rope ? 2 : 4; }
// Calls that overlap on one workspace are an error of the caller: one call clears the other's words, or leaves anything at all
// in them where the shapes differ.  Their results are undefined, but every access stays in the pot and their kernels end: a
// ticket counts only if it names a chunk of this call, a workgroup takes no more of them than there are chunks, and its waits
// for smaller chunks, which take microseconds, are bounded (seconds in all).
constexpr int kMarkPolls = 1 << 22;
// ... SHARED (half with ROPE, whose coefficients take as many registers again): at most 64 KiB of each tensor per workgroup
constexpr int sh_unroll(int threads, bool rope) { return 4096 / threads / (rope ? 2 : 1); }

__device__ __forceinline__ uint32_t agent_load(const uint32_t* p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ uint32_t agent_add(uint32_t* p, uint32_t v) {
  return __hip_atomic_fetch_add(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// ROPE (CR-RoPE, Sec. 3.5): the kernel also writes Krot[j] = rotary embedding at position j of the kept key j, for all
// j < k (rows that stay where they are included, so every kept K row is read); the pot itself keeps the plain keys.
// ROWB, BF16: row bytes and cache type where ROPE needs them at compile time (ROWB is 0 without: `row_shift` = log2 of the
// 16-byte lanes of a row).
// NUC (SHARED, rows of up to kNoveltyMaxRow tokens): the unit's words say which tokens have a NuC slot.  (In one kernel with the way that finds
// them, calls without paid for it: 80 units of 2912 tokens 96.7 -> 97.4 us, 84 of 896 fp32 tokens 100.0 -> 101.0.)
template <int THREADS, int CH, int ROWB, bool BF16, bool SHARED, bool NUC>
__global__ __launch_bounds__(THREADS, sc_min_waves(SHARED, CH, ROWB)) void select_compact_kernel(Dims D, const float* __restrict__ u,
                                                                     float* novelty, int carry_novelty, float* scores,
                                                                     int32_t* __restrict__ keep_idx, char* Kbuf,
                                                                     char* Vbuf, const float* __restrict__ rope_cos,
                                                                     const float* __restrict__ rope_sin, char* Krot,
                                                                     int row_shift, int wgs_per_unit, int chunks,
                                                                     int chunk_rows, uint32_t* sync) {
  constexpr bool ROPE = ROWB > 0;
  constexpr bool kRegs = RowStore<THREADS, CH>::kRegs;
  __shared__ SelectShared<THREADS, CH> sh;
  // The kept list: in LDS for short rows; a long row leaves no room for it, and it is read back from keep_idx, where this
  // workgroup has just put it
  __shared__ uint16_t keep_lds[kRegs ? CH * 4 * THREADS : 1];
  __shared__ uint32_t ticket_lds;
  __shared__ int last_lds;
  const int part = SHARED ? blockIdx.x % wgs_per_unit : 0;
  const int unit = D.unit0 + (SHARED ? blockIdx.x / wgs_per_unit : blockIdx.x);
  const UnitIdx ui = decode_unit(D, unit);
  uint32_t* sy = SHARED ? sync + (int64_t)unit * kSyncWords : nullptr;
  if (SHARED && threadIdx.x == 0) ticket_lds = agent_add(&sy[kSyncTicket], 1u) & 0xFFFFu;
  int32_t* keep_out = keep_idx + (int64_t)unit * D.k;
  float* nov = (D.T > 0 || carry_novelty) ? novelty + nov_offset(D, ui) : nullptr;
  {
    Row<THREADS, CH> row(D, sh, unit, u, nullptr, nov);
    const uint32_t* nuc_words = NUC ? sync + (int64_t)novelty_unit(D, unit) * kSyncWords : nullptr;
    select_row<THREADS, CH, true, NUC>(row, part == 0 && scores != nullptr ? scores + (int64_t)unit * D.n : nullptr, nuc_words,
                         [&](int pos, int t, int c, int i) {
                           if (kRegs) keep_lds[pos] = (uint16_t)t;
                           else       keep_out[pos] = t;
                           // carried novelty moves up with the rows: every thread has had its entries in registers
                           // since before the barriers of the selection
                           if constexpr (kRegs && !SHARED) { if (carry_novelty) nov[pos] = row.nv[4 * c + i]; }
                         });
  }
  __syncthreads();
  auto keep = [&](int j) { return kRegs ? (int)keep_lds[j] : min(max(keep_out[j], 0), D.n - 1); };
  if (kRegs && part == 0)
    for (int j = threadIdx.x; j < D.k; j += THREADS) keep_out[j] = keep_lds[j];
  // (keep[j] >= j: a chunk's sources are read before anything at or above them is written)
  auto compact_novelty = [&]() {
    constexpr int kN = 8;
    for (int base = 0; base < D.k; base += kN * THREADS) {
      float v[kN];
      int sidx[kN];
#pragma unroll
      for (int i = 0; i < kN; ++i) sidx[i] = keep(min(base + i * THREADS + (int)threadIdx.x, D.k - 1));
      arrived(sidx);
#pragma unroll
      for (int i = 0; i < kN; ++i) {
        const int j = base + i * THREADS + threadIdx.x;
        if (j < D.k) v[i] = nov[sidx[i]];
      }
      wait_for_loads();
      __syncthreads();
#pragma unroll
      for (int i = 0; i < kN; ++i) {
        const int j = base + i * THREADS + threadIdx.x;
        if (j < D.k) nov[j] = v[i];
      }
    }
  };
  if constexpr (!kRegs && !SHARED) { if (carry_novelty) compact_novelty(); }

  const int rowb = ROPE ? ROWB : 16 << row_shift;
  const int64_t ubytes = kv_offset(D, ui) * (int64_t)(D.dtype == 0 ? 4 : 2);
  const int half_d = D.d / 2;
  const int lane_shift = ROPE ? __ffs(ROWB / 16) - 1 : row_shift;
  char* kb = Kbuf + ubytes;
  char* vb = Vbuf + ubytes;
  char* rb = ROPE ? Krot + ubytes : nullptr;
  const int lane_in_row = threadIdx.x & ((1 << lane_shift) - 1);
  const int lane_off = lane_in_row * 16;
  const int row_in_pass = threadIdx.x >> lane_shift, rows_per_pass = THREADS >> lane_shift;
  constexpr int kUnroll = !SHARED ? sc_unroll(ROPE) : sh_unroll(THREADS, ROPE);

  if (SHARED && carry_novelty && threadIdx.x == 0)
    last_lds = agent_add(&sy[kSyncTicket], kSyncOneSelected) >> 16 == (uint32_t)(wgs_per_unit - 1);
  uint32_t ticket = SHARED ? ticket_lds : 0u;
  int base = SHARED ? chunk_first_row(ticket, chunks, chunk_rows, D.k) : 0;
  int taken = 0, polls = kMarkPolls;
  while (base < D.k) {
    const int end = SHARED ? min(D.k, base + chunk_rows) : D.k;
    uint4 a[kUnroll], b[kUnroll];
    bool move[kUnroll];
    RopeCoef<ROPE ? ROWB : 128, BF16> coef[ROPE ? kUnroll : 1];
    int sidx[kUnroll];                            // ascending, in [j, n)
#pragma unroll
    for (int i = 0; i < kUnroll; ++i) sidx[i] = keep(min(base + i * rows_per_pass + row_in_pass, end - 1));
    arrived(sidx);
#pragma unroll
    for (int i = 0; i < kUnroll; ++i) {
      const int j = base + i * rows_per_pass + row_in_pass;
      move[i] = false;
      if (j < end) {
        move[i] = sidx[i] != j;
        if (move[i] || ROPE) a[i] = load_streaming(kb + (int64_t)sidx[i] * rowb + lane_off);
        if (move[i]) b[i] = load_streaming(vb + (int64_t)sidx[i] * rowb + lane_off);
        if constexpr (ROPE) coef[i].load(lane_in_row, rope_cos + (int64_t)j * half_d, rope_sin + (int64_t)j * half_d);
      }
    }
    // (one workgroup per unit with CR-RoPE: with all loads in flight at once 160 units of 2500 tokens went 189 -> 192 us, 256 to 640 units
    // stayed the same)
    if constexpr (ROPE && !SHARED) asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    else wait_for_loads();
    __syncthreads();
    int next = base + kUnroll * rows_per_pass;
    if constexpr (SHARED) {
      if (threadIdx.x < 64) {
        const int chunk = (int)ticket, lane = threadIdx.x;
        if (lane == 0) {
          __hip_atomic_fetch_or(&sy[kSyncMarks + chunk / 32], 1u << (chunk % 32), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
          ticket_lds = agent_add(&sy[kSyncTicket], 1u) & 0xFFFFu;
        }
        const int below = chunk - 32 * lane;      // chunks before this one that lane's word of marks holds
        const uint32_t want = below >= 32 ? 0xFFFFFFFFu : (below > 0 ? (1u << below) - 1u : 0u);
        const uint32_t* word = &sy[kSyncMarks + min(lane, kSyncMarkWords - 1)];
        for (; polls > 0 && !__all((want & ~agent_load(word)) == 0u); --polls) __builtin_amdgcn_s_sleep(1);
      }
      __syncthreads();
      ticket = ticket_lds;
      next = ++taken < chunks ? chunk_first_row(ticket, chunks, chunk_rows, D.k) : D.k;
    }
#pragma unroll
    for (int i = 0; i < kUnroll; ++i) {
      const int j = base + i * rows_per_pass + row_in_pass;
      if (move[i]) {
        store_streaming(kb + (int64_t)j * rowb + lane_off, a[i]);
        store_streaming(vb + (int64_t)j * rowb + lane_off, b[i]);
      }
      if constexpr (ROPE) {
        if (j < end)
          store_streaming(rb + (int64_t)j * rowb + lane_off, rope_lane<ROWB, BF16>(a[i], lane_in_row, coef[i]));
      }
    }
    base = next;
  }
  if constexpr (SHARED) {
    // all workgroups of the unit have read the novelty they select by once the last one has selected
    if (carry_novelty) {
      __syncthreads();
      if (last_lds) compact_novelty();
    }
  }
}

// Stand-alone CR-RoPE: Krot[j] = rotary embedding at position j of K[j], j < count, for every unit of the launch.
// A thread handles kRopeUnroll rows (all their loads in flight together).
constexpr int kRopeUnroll = 4;

template <int ROWB, bool BF16>
__global__ __launch_bounds__(256) void rope_rows_kernel(Dims D, const char* __restrict__ Kbuf,
                                                        const float* __restrict__ rope_cos,
                                                        const float* __restrict__ rope_sin, int count, char* Krot) {
  constexpr int kLanesPerRow = ROWB / 16;
  constexpr int kRowsPerPass = 256 / kLanesPerRow;
  constexpr int kRowsPerBlock = kRowsPerPass * kRopeUnroll;
  const int blocks_per_unit = (count + kRowsPerBlock - 1) / kRowsPerBlock;
  const int unit = D.unit0 + blockIdx.x / blocks_per_unit;
  const int64_t ubytes = kv_offset(D, decode_unit(D, unit)) * (int64_t)(ROWB / D.d);
  const int lane_in_row = threadIdx.x % kLanesPerRow;
  const int j0 = (blockIdx.x % blocks_per_unit) * kRowsPerBlock + threadIdx.x / kLanesPerRow;
  const int half_d = D.d / 2;
  uint4 x[kRopeUnroll];
  RopeCoef<ROWB, BF16> coef[kRopeUnroll];
#pragma unroll
  for (int i = 0; i < kRopeUnroll; ++i) {
    const int j = j0 + i * kRowsPerPass;
    if (j < count) {                                           // whole rows: both lanes of a pair agree
      x[i] = load_streaming(Kbuf + ubytes + (int64_t)j * ROWB + lane_in_row * 16);
      coef[i].load(lane_in_row, rope_cos + (int64_t)j * half_d, rope_sin + (int64_t)j * half_d);
    }
  }
#pragma unroll
  for (int i = 0; i < kRopeUnroll; ++i) {
    const int j = j0 + i * kRowsPerPass;
    if (j < count)
      store_streaming(Krot + ubytes + (int64_t)j * ROWB + lane_in_row * 16, rope_lane<ROWB, BF16>(x[i], lane_in_row, coef[i]));
  }
}

}  // namespace

bool select_compact_supported(const Dims& D) { return D.n <= kLdsRowTokens; }

// Several workgroups per unit as long as there is a compute unit for each, in chunks of at least one and at most
// sh_unroll rows per thread; 32 marks per word bound the number of chunks.
// A call with more chunks than workgroups has the largest ones.  The last word of marks, which holds something else where slots are found
// beside the scores, is therefore only reached by calls that keep more than kNoveltyMaxKept tokens:
constexpr int largest_chunk(int threads) { return (threads >> 5) * sh_unroll(threads, true); }         // rows of 512 bytes, CR-RoPE
static_assert(std::min(largest_chunk(512), largest_chunk(1024)) * 32 * (kSyncMarkWords - 1) >= kNoveltyMaxKept, "");
static_assert(kSharedFillWorkgroups <= 32 * (kSyncMarkWords - 1), "");
static int log2_row_lanes(const Dims& D) { return (D.d == 128 ? 4 : 3) + (D.dtype == 0 ? 1 : 0); }      // 16-byte lanes of a row
struct SharedCut { int per_unit, chunk_rows; };            // (one workgroup per unit: not shared)
static SharedCut shared_cut(const Dims& D, bool rope) {
  const int threads = sc_threads(true, D.n), rows_per_pass = threads >> log2_row_lanes(D);
  const int max_rows = rows_per_pass * sh_unroll(threads, rope);
  const int per_unit = std::min(kSharedFillWorkgroups / std::max(D.units_run, 1), (D.k + rows_per_pass - 1) / rows_per_pass);
  if (per_unit <= 1) return {1, 0};
  const int rows = std::min((D.k + per_unit - 1) / per_unit, max_rows);
  const int chunk_rows = (rows + rows_per_pass - 1) / rows_per_pass * rows_per_pass;
  if (D.k > chunk_rows * 32 * kSyncMarkWords) return {1, 0};
  return {std::min(per_unit, (D.k + chunk_rows - 1) / chunk_rows), chunk_rows};
}
bool select_compact_shares_units(const Dims& D, bool rope) { return shared_cut(D, rope).per_unit > 1; }

// pooling + NuC lift + top-k + in-place compaction of K and V (and of carried per-head novelty).
// Krot != nullptr: CR-RoPE of the kept keys on the side (rope_cos / rope_sin: [>= k, d/2] fp32).
// sync: kSyncWords words per unit, as the first score kernel of the call leaves them; null for more than kMaxSharedUnits units.
void launch_select_compact(const Dims& D, const float* u, float* novelty, bool carry_novelty, float* scores,
                           int32_t* keep_idx, void* K, void* V, const float* rope_cos, const float* rope_sin, void* Krot,
                           uint32_t* sync, bool nuc_known, hipStream_t s) {
  const int rowb = D.d * (D.dtype == 0 ? 4 : 2), row_shift = log2_row_lanes(D);
  const SharedCut cut = shared_cut(D, Krot != nullptr);
  const int per_unit = cut.per_unit, chunk_rows = cut.chunk_rows;
  const bool shared = per_unit > 1;
  const int chunks = shared ? (D.k + chunk_rows - 1) / chunk_rows : 0;
  const int threads = sc_threads(shared, D.n);
  const dim3 grid((unsigned)D.units_run * per_unit), block(threads);
#define CCD_LAUNCH(THREADS, CH, RB, BF, SHARED, NUC)                                                                                  \
  launch((select_compact_kernel<THREADS, CH, RB, BF, SHARED, NUC>), grid, block, s, D, u, novelty, carry_novelty ? 1 : 0, scores,       \
         keep_idx, (char*)K, (char*)V, rope_cos, rope_sin, (char*)Krot, row_shift, per_unit, chunks, chunk_rows, sync)
#define CCD_LAUNCH_RB(THREADS, CH, SHARED, NUC)                                          \
  if (Krot == nullptr) CCD_LAUNCH(THREADS, CH, 0, true, SHARED, NUC);                    \
  else if (rowb == 128) CCD_LAUNCH(THREADS, CH, 128, true, SHARED, NUC);                 \
  else if (rowb == 256 && D.dtype == 1) CCD_LAUNCH(THREADS, CH, 256, true, SHARED, NUC); \
  else if (rowb == 256) CCD_LAUNCH(THREADS, CH, 256, false, SHARED, NUC);                \
  else CCD_LAUNCH(THREADS, CH, 512, false, SHARED, NUC)
#define CCD_LAUNCH_SHARED(CH) \
  if (shared) { CCD_LAUNCH_RB(1024, CH, true, false); } else { CCD_LAUNCH_RB(1024, CH, false, false); }
#define CCD_LAUNCH_NUC(THREADS, CH)          /* rows of up to kNoveltyMaxRow tokens */ \
  if (nuc_known) { CCD_LAUNCH_RB(THREADS, CH, true, true); } else { CCD_LAUNCH_RB(THREADS, CH, true, false); }
  static_assert(kNoveltyMaxRow <= 2 * 4 * 1024, "");
  const int token_chunks = (D.n + 4 * threads - 1) / (4 * threads);     // per thread
  if (threads == 512)         { if (token_chunks <= 1) { CCD_LAUNCH_NUC(512, 1); } else { CCD_LAUNCH_NUC(512, 2); } }
  else if (token_chunks <= 1) { CCD_LAUNCH_RB(1024, 1, false, false); }
  else if (token_chunks <= 2) { if (shared) { CCD_LAUNCH_NUC(1024, 2); } else { CCD_LAUNCH_RB(1024, 2, false, false); } }
  else if (token_chunks <= 4 && shared) { CCD_LAUNCH_RB(1024, 4, true, false); }
  else                        { CCD_LAUNCH_SHARED(kLdsRow); }
#undef CCD_LAUNCH_SHARED
#undef CCD_LAUNCH_NUC
#undef CCD_LAUNCH_RB
#undef CCD_LAUNCH
}

void launch_rope_rows(const Dims& D, const void* K, const float* rope_cos, const float* rope_sin, int count, void* Krot,
                      hipStream_t s) {
  const int rowb = D.d * (D.dtype == 0 ? 4 : 2);
  const int rows_per_block = 256 / (rowb / 16) * kRopeUnroll;
  const dim3 grid((unsigned)((count + rows_per_block - 1) / rows_per_block) * (unsigned)D.units_run), block(256);
#define CCD_LAUNCH(RB, BF) \
  launch((rope_rows_kernel<RB, BF>), grid, block, s, D, (const char*)K, rope_cos, rope_sin, count, (char*)Krot)
  if (rowb == 128) CCD_LAUNCH(128, true);
  else if (rowb == 256 && D.dtype == 1) CCD_LAUNCH(256, true);
  else if (rowb == 256) CCD_LAUNCH(256, false);
  else CCD_LAUNCH(512, false);
#undef CCD_LAUNCH
}

void launch_append(const Dims& D, int count, void* K, void* V, const void* K_new, const void* V_new, float* novelty,
                   const float* novelty_new, bool nov_per_head, hipStream_t s) {
  const int esz = D.dtype == 0 ? 4 : 2;
  const int64_t run = (int64_t)count * D.d * esz;
  const int segs = (int)((run + kApSegBytes - 1) / kApSegBytes);
  // (a grid has fewer than 2^32 threads: millions of units go in several launches)
  const int64_t most = std::max<int64_t>(1, ((int64_t)1 << 31) / ((int64_t)2 * segs * kApThreads));
  const bool values_first = 4 * D.units * run >= kMemorySideCache;
  Dims R = D;
  const int64_t all_segs = (D.units * run + kApSegBytes - 1) / kApSegBytes;
  const bool dense = D.kv_sh == (int64_t)D.n_cap * D.d && (D.L == 1 || D.kv_sl == D.Hkv * D.kv_sh) && (D.B == 1 || D.kv_sb == D.L * D.Hkv * D.kv_sh);
  if (values_first && D.n == 0 && count == D.n_cap && dense && run > kApSegBytes && run % kApSegBytes != 0 && 2 * all_segs * kApThreads <= (int64_t)1 << 31) {
    // (units of more than a segment: there are no fewer segments than pieces of novelty; of whole segments: the cut is the same either way)
    const int64_t pieces = (int64_t)(nov_per_head ? D.units : D.B) * ((count + kApNovelty - 1) / kApNovelty);
    launch(append_rows_kernel<true>, dim3(2u * (unsigned)all_segs), dim3(kApThreads), s, R, esz, count, (int)all_segs, (char*)K, (char*)V,
           (const char*)K_new, (const char*)V_new, novelty, novelty_new, nov_per_head ? 1 : 0, 1, (int)(all_segs / pieces));
    return;
  }
  for (int64_t u0 = 0; u0 < D.units; u0 += most) {
    R.unit0 = (int)u0;
    R.units_run = (int)std::min<int64_t>(most, D.units - u0);
    launch(append_rows_kernel<false>, dim3(2u * R.units_run * segs), dim3(kApThreads), s, R, esz, count, segs, (char*)K, (char*)V,
           (const char*)K_new, (const char*)V_new, novelty, novelty_new, nov_per_head ? 1 : 0, values_first ? 1 : 0, 0);
  }
}

void launch_compact(const Dims& D, const void* Ksrc, const void* Vsrc, const int32_t* keep_idx, void* Kdst, void* Vdst,
                    float* novelty, hipStream_t s) {
  const int rowb = D.d * (D.dtype == 0 ? 4 : 2);
  const dim3 grid(2u * D.units_run), block(kCpThreads);
  const int seg_rows = kGaThreads / (rowb / 16) * kGaRows, segs = (D.k + seg_rows - 1) / seg_rows;
  // (a grid has fewer than 2^32 threads)
  const bool gather = Ksrc != Kdst && Vsrc != Vdst && (int64_t)D.units_run * segs * 2 * kGaThreads <= (int64_t)1 << 31;
#define CCD_LAUNCH(RB)                                                                                              \
  if (gather)                                                                                                       \
    launch((gather_rows_kernel<RB>), dim3(2u * D.units_run * segs), dim3(kGaThreads), s, D, segs, (const char*)Ksrc, \
           (const char*)Vsrc, keep_idx, (char*)Kdst, (char*)Vdst);                                                  \
  else                                                                                                              \
    launch((compact_rows_kernel<RB>), grid, block, s, D, (const char*)Ksrc, (const char*)Vsrc, keep_idx, (char*)Kdst, (char*)Vdst)
  if (rowb == 128) { CCD_LAUNCH(128); }
  else if (rowb == 256) { CCD_LAUNCH(256); }
  else { CCD_LAUNCH(512); }
#undef CCD_LAUNCH
  if (novelty != nullptr)
    launch(compact_novelty_kernel, dim3(D.units_run), block, s, D, keep_idx, novelty);
}

}  // namespace ccd
