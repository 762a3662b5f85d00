// Gather-only lookup kernel for gfx950 (MI355X): the GM data flow of Sec. II-B (rows
// straight from HBM) with sum / mean pooling, for plans whose slices are all GATHER and
// whose rows are 256, 512 or 1024 bytes wide (G = 16, 32 or 64 lanes of 16 bytes).
//
// The unit of work is a wavefront, and every decision it takes is wave-uniform: which
// chunk of bags it walks, where a step starts and ends, where each bag ends.  So the
// control lives in scalar registers and the vector registers hold only row data, the
// accumulators and one index per lane (86-118 VGPRs with kSteps = 12-16 rows in flight
// per SW: one 1024-thread workgroup per CU, 4 wavefronts per SIMD; measured, 12 in flight
// at that occupancy beats 6 or 8 at two workgroups per CU).  The file is built once per
// kSteps (EMBX_GKS = 12, 13, 16) and a plan picks the one whose steps its chunks fill best.
//
// What bounds it: instruction issue on short bags; on long ones the bytes beyond L2 (131M
// lookups of 512-byte rows: 18.8 GB at 97% of a copy's rate, 3.80 ms) and close behind them the
// vector memory pipe (its address unit is busy 88% of that time; with every row an L2 hit the
// batch takes 2.84 ms); and HBM writes of the pooled rows (without them, 3.4M fp16 lookups of
// 256 bytes would take 64 us, not 105).  Hence scalar control that costs three instructions per
// row load (see Multi).
//
// A wavefront is S = 64 / G sub-wavefronts (SWs) of G lanes; lane i of a SW covers bytes
// [16 i, 16 i + 16) of a row.  A step covers N = S * kSteps consecutive lookups of the
// current chunk: instruction u loads lookups p + u S + s (s = the SW), one row per SW,
// with a structured buffer load (the hardware forms table + row * R + 16 i from the row
// number, so a lookup costs no address arithmetic).  Lane 16 r + u of SW s's rows loads
// the id of lookup u S + s, and one DPP row broadcast hands it to every lane of the SW.
// Each SW adds its own lookups; where a bag ends (a position known to the whole
// wavefront), the S partial sums are combined by a reduce-scatter across the SWs
// (v_permlane32_swap between the wavefront's halves, v_permlane16_swap between
// neighbouring rows of 16 lanes), after which each lane holds E / 64 of the bag's sums
// and the whole wavefront stores the pooled row once.  The additions of a bag follow
// from the plan and the batch alone, so results are bitwise reproducible.
//
// Bags of tables whose statistics promise at most one lookup per bag are a second
// queue: a step covers N bags, each SW loads one bag's row and stores it as the bag's
// output (no reduction); a bag that holds more lookups at run time is summed on a slow
// path, so any batch stays correct.
//
// An id outside [0, rows) adds nothing: it is counted, and its load goes past the table's
// descriptor, which returns zeros without an access (tables of 4 GiB or more, read with
// 64-bit addresses, load row 0 and clear it).
#include <hip/hip_fp16.h>
#include <hip/hip_runtime.h>

#include <utility>

#include "device_types.hpp"
#include "positions.hpp"

#ifndef EMBX_GPART
#define EMBX_GPART -1
#endif
#ifndef EMBX_GKS
#define EMBX_GKS 12
#endif
#define EMBX_HAS_GPART(p) (EMBX_GPART < 0 || EMBX_GPART == (p))

#if defined(__HIP_DEVICE_COMPILE__)
#define GMEM __attribute__((address_space(1)))
#define LMEM __attribute__((address_space(3)))
#else
#define GMEM
#define LMEM
#endif

namespace embx {

typedef int i32x4 __attribute__((ext_vector_type(4)));

// structured buffer load of 16 bytes: base + vindex * stride + voffset (buffer descriptor
// in scalar registers; an access past num_records reads zeros)
__device__ i32x4 buffer_load_row(i32x4 rsrc, int vindex, int voffset, int soffset, int aux)
    __asm("llvm.amdgcn.struct.buffer.load.v4i32");

typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x2 __attribute__((ext_vector_type(2)));

// raw buffer stores: base + voffset, dropped where voffset runs past num_records
__device__ void buffer_store_f32(float v, i32x4 rsrc, int voffset, int soffset, int aux)
    __asm("llvm.amdgcn.raw.buffer.store.f32");
__device__ void buffer_store_f32x2(f32x2 v, i32x4 rsrc, int voffset, int soffset, int aux)
    __asm("llvm.amdgcn.raw.buffer.store.v2f32");
__device__ void buffer_store_f32x4(f32x4 v, i32x4 rsrc, int voffset, int soffset, int aux)
    __asm("llvm.amdgcn.raw.buffer.store.v4f32");

namespace {

typedef unsigned u32x4 __attribute__((ext_vector_type(4)));

constexpr int kSteps = EMBX_GKS;   // row loads in flight per lane per step (one build per value)
static_assert(kSteps >= 1 && kSteps <= 16, "one id per lane of a row of 16 for each step");

// f(integral_constant<int, 0>), ..., f(integral_constant<int, N - 1>): a loop whose index
// is a compile-time constant (register arrays stay in registers, DPP controls are immediates)
template <class F, int... I>
__device__ __forceinline__ void static_for_impl(F&& f, std::integer_sequence<int, I...>) {
  (f(std::integral_constant<int, I>{}), ...);
}
template <int N, class F>
__device__ __forceinline__ void static_for(F&& f) {
  static_for_impl(f, std::make_integer_sequence<int, N>{});
}

// Buffer descriptor of a table: rows of R bytes from base; num_records = rows (the
// structured range check compares the row index).  Configuration dword for gfx9:
// 32-bit data format, everything else zero.
__device__ __forceinline__ i32x4 table_rsrc(const void* base, int R, uint32_t rows) {
  const uint64_t b = reinterpret_cast<uint64_t>(base);
  i32x4 d;
  d.x = __builtin_amdgcn_readfirstlane(static_cast<int>(b & 0xffffffffu));
  d.y = __builtin_amdgcn_readfirstlane(static_cast<int>(((b >> 32) & 0xffffu) | (static_cast<uint32_t>(R) << 16)));
  d.z = __builtin_amdgcn_readfirstlane(static_cast<int>(rows));
  d.w = 0x00020000;
  return d;
}

// lane u of this lane's row of 16 (DPP row_newbcast:u)
template <int U>
__device__ __forceinline__ int row_bcast(int v) {
  return __builtin_amdgcn_mov_dpp(v, 0x150 + U, 0xF, 0xF, true);
}

// a value that is the same in every lane, kept in scalar registers
__device__ __forceinline__ int uni(int v) { return __builtin_amdgcn_readfirstlane(v); }
__device__ __forceinline__ int64_t uni64(int64_t v) {
  const int lo = __builtin_amdgcn_readfirstlane(static_cast<int>(v & 0xffffffff));
  const int hi = __builtin_amdgcn_readfirstlane(static_cast<int>(v >> 32));
  return (static_cast<int64_t>(hi) << 32) | static_cast<uint32_t>(lo);
}

// Waits for every memory operation in flight; the empty asm keeps the compiler from
// moving loads across the wait.
__device__ __forceinline__ void wait_all() {
  asm volatile("" ::: "memory");
  __builtin_amdgcn_s_waitcnt(0);
}

template <bool F16>
struct Acc {
  static constexpr int NA = F16 ? 8 : 4;
  float v[NA];
};

template <bool F16>
__device__ __forceinline__ void acc_zero(Acc<F16>& a) {
#pragma unroll
  for (int i = 0; i < Acc<F16>::NA; ++i) a.v[i] = 0.0f;
}

// x * wt + acc, one rounding per element (wt = the weight, or a run-time 1: then the
// result is the plain sum bit for bit); fp16 halves take one mixed-precision fma each
__device__ __forceinline__ void acc_add(Acc<false>& a, const i32x4 r, float wt) {
  a.v[0] = __builtin_fmaf(__int_as_float(r.x), wt, a.v[0]);
  a.v[1] = __builtin_fmaf(__int_as_float(r.y), wt, a.v[1]);
  a.v[2] = __builtin_fmaf(__int_as_float(r.z), wt, a.v[2]);
  a.v[3] = __builtin_fmaf(__int_as_float(r.w), wt, a.v[3]);
}

__device__ __forceinline__ float half_lo(int w) {
  return __half2float(__ushort_as_half(static_cast<unsigned short>(static_cast<uint32_t>(w) & 0xffffu)));
}
__device__ __forceinline__ float half_hi(int w) {
  return __half2float(__ushort_as_half(static_cast<unsigned short>(static_cast<uint32_t>(w) >> 16)));
}

__device__ __forceinline__ void acc_add(Acc<true>& a, const i32x4 r, float wt) {
  const int w[4] = {r.x, r.y, r.z, r.w};
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    a.v[2 * q] = __builtin_fmaf(half_lo(w[q]), wt, a.v[2 * q]);
    a.v[2 * q + 1] = __builtin_fmaf(half_hi(w[q]), wt, a.v[2 * q + 1]);
  }
}

__device__ __forceinline__ i32x4 zero4() { return i32x4{0, 0, 0, 0}; }

template <class T>
__device__ __forceinline__ GMEM T* as_global(T* p) {
  return (GMEM T*)p;
}

// Reduce-scatter of the S partial sums of a wavefront: afterwards a[0 .. NA/S) of a lane
// of SW s hold elements [s NA/S, (s+1) NA/S) of its 16-byte piece, summed over the SWs
// (halves first: SW s + S/2 onto SW s; then neighbouring rows).  Fixed order.
template <int S, int NA>
__device__ __forceinline__ void reduce_scatter(float (&a)[NA]) {
  if constexpr (S >= 2) {
#pragma unroll
    for (int i = 0; i < NA / 2; ++i) {
      const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(a[i]), __float_as_uint(a[i + NA / 2]), false,
                                                       false);
      a[i] = __uint_as_float(r[0]) + __uint_as_float(r[1]);
    }
  }
  if constexpr (S >= 4) {
#pragma unroll
    for (int i = 0; i < NA / 4; ++i) {
      const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(a[i]), __float_as_uint(a[i + NA / 4]), false,
                                                       false);
      a[i] = __uint_as_float(r[0]) + __uint_as_float(r[1]);
    }
  }
}

// non-temporal store of P floats (pooled outputs are not read again by the launch)
template <int P>
__device__ __forceinline__ void store_part(GMEM float* q, const float* v) {
  if constexpr (P == 4) {
    const f32x4 x = {v[0], v[1], v[2], v[3]};
    __builtin_nontemporal_store(x, reinterpret_cast<GMEM f32x4*>(q));
  } else if constexpr (P == 8) {
    const f32x4 x = {v[0], v[1], v[2], v[3]};
    const f32x4 y = {v[4], v[5], v[6], v[7]};
    __builtin_nontemporal_store(x, reinterpret_cast<GMEM f32x4*>(q));
    __builtin_nontemporal_store(y, reinterpret_cast<GMEM f32x4*>(q + 4));
  } else if constexpr (P == 2) {
    const f32x2 x = {v[0], v[1]};
    __builtin_nontemporal_store(x, reinterpret_cast<GMEM f32x2*>(q));
  } else {
    static_assert(P == 1, "part size");
    __builtin_nontemporal_store(v[0], q);
  }
}

// The same through a descriptor of the pooled row, which drops what lies past its end (the
// lanes of a row narrower than its sub-wavefront): a store without a branch.
constexpr int kNonTemporal = 2;
template <int P>
__device__ __forceinline__ void buffer_store_part(i32x4 rsrc, int off, const float* v) {
  if constexpr (P >= 4) {
#pragma unroll
    for (int i = 0; i < P; i += 4)
      buffer_store_f32x4(f32x4{v[i], v[i + 1], v[i + 2], v[i + 3]}, rsrc, off + 4 * i, 0, kNonTemporal);
  } else if constexpr (P == 2) {
    buffer_store_f32x2(f32x2{v[0], v[1]}, rsrc, off, 0, kNonTemporal);
  } else {
    static_assert(P == 1, "part size");
    buffer_store_f32(v[0], rsrc, off, 0, kNonTemporal);
  }
}

// A gather run in LDS (see GatherRun; its j and k hold the slice's first and end bag at the
// runtime batch there): chunk c of a queue is bags [bs + (c - chunk_base) cb, + cb) of the
// slice, clipped to it.
struct Chunk {
  int run;      // record in the worker's LDS slot, -1 = none
  int bs, be;   // bags
};

// The chunks of one queue of the worker, claimed by wavefronts: wavefront v first takes
// chunk v, then further chunks in order from a counter in LDS.
struct WaveQueue {
  const LMEM GatherRun* r;
  int e, e_end, nchunks;
  LMEM int* ctr;
  int first;    // this wavefront's first chunk, -1 once taken
  int waves;    // wavefronts of the worker
  __device__ __forceinline__ int claim() {
    if (first >= 0) {
      const int v = first;
      first = -1;
      return v;
    }
    if (nchunks <= waves) return nchunks;
    int v = 0;
    if ((threadIdx.x & 63) == 0) v = atomicAdd(ctr, 1);
    return __builtin_amdgcn_readfirstlane(v);   // lane 0 (every lane is active here)
  }
  __device__ __forceinline__ Chunk next() {
    while (true) {
      const int c = claim();
      if (c >= nchunks) return Chunk{-1, 0, 0};
      // the run holding chunk c: chunk_base ascends, so count the runs after e that start at or before c
      while (true) {
        const int x = e + 1 + static_cast<int>(threadIdx.x & 63);
        const int passed = __popcll(__ballot(x < e_end && r[min(x, e_end - 1)].chunk_base <= c));
        e = uni(e + passed);
        if (passed < 64) break;
      }
      const int bs = __builtin_amdgcn_readfirstlane(r[e].j), be = __builtin_amdgcn_readfirstlane(r[e].k);
      const int cb = __builtin_amdgcn_readfirstlane(r[e].cb);
      const int c0b = __builtin_amdgcn_readfirstlane(r[e].chunk_base);
      const int c0 = bs + (c - c0b) * cb;
      const int c1 = min(be, c0 + cb);
      if (c0 < c1) return Chunk{uni(e), uni(c0), uni(c1)};
    }
  }
};

// Per-chunk constants of a table, wave-uniform: the buffer descriptor of its rows (base,
// stride R, num_records = rows), the table id and flags.  Tables of 4 GiB or more are read
// with 64-bit addresses (the buffer unit's offset arithmetic is 32 bits wide).
struct RunInfo {
  i32x4 rsrc;
  int table;
  int flags;   // bit 0: mean pooling; bit 1: rows * R >= 2^32
  __device__ __forceinline__ uint64_t rows() const { return static_cast<uint32_t>(rsrc.z); }
  __device__ __forceinline__ bool mean() const { return (flags & 1) != 0; }
  __device__ __forceinline__ bool big() const { return (flags & 2) != 0; }
  __device__ __forceinline__ GMEM const char* base() const {
    const uint64_t b = (static_cast<uint64_t>(static_cast<uint32_t>(rsrc.y) & 0xffffu) << 32) |
                       static_cast<uint32_t>(rsrc.x);
    return (GMEM const char*)b;
  }
};

#define CMEM __attribute__((address_space(4)))

__device__ __forceinline__ RunInfo run_info(const LMEM GatherRun* runs, int e, const LookupArgs& a) {
  const LMEM GatherRun& g = runs[e];
  const uint64_t w = (static_cast<uint64_t>(static_cast<uint32_t>(__builtin_amdgcn_readfirstlane(
                          static_cast<int>(reinterpret_cast<uint64_t>(g.w) >> 32)))) << 32) |
                     static_cast<uint32_t>(__builtin_amdgcn_readfirstlane(
                         static_cast<int>(reinterpret_cast<uint64_t>(g.w) & 0xffffffffu)));
  const uint32_t rows = static_cast<uint32_t>(__builtin_amdgcn_readfirstlane(static_cast<int>(g.rows & 0xffffffff)));
  RunInfo ri;
  ri.rsrc = table_rsrc(reinterpret_cast<const void*>(w), a.R, rows);
  ri.table = __builtin_amdgcn_readfirstlane(g.table);
  ri.flags = (__builtin_amdgcn_readfirstlane(g.mean) != 0 ? 1 : 0) |
             (static_cast<uint64_t>(rows) * static_cast<uint64_t>(a.R) >= (uint64_t(1) << 32) ? 2 : 0);
  return ri;
}

// row `row` of the table, this lane's 16 bytes (lane_c: byte offset in the row)
__device__ __forceinline__ i32x4 load_row(const RunInfo& ri, int row, int lane_c, int R) {
  if (ri.big())
    return *reinterpret_cast<GMEM const i32x4*>(ri.base() +
                                                static_cast<uint64_t>(static_cast<uint32_t>(row)) * static_cast<uint32_t>(R) +
                                                lane_c);
  return buffer_load_row(ri.rsrc, row, lane_c, 0, 0);
}

// registers that hold nothing (so that what an earlier step left in them is not kept)
template <int U>
__device__ __forceinline__ void undefined_rows(i32x4 (&raw)[kSteps]) {
  if constexpr (U < kSteps) {
    asm volatile("" : "=v"(raw[U]));
    undefined_rows<U + 1>(raw);
  }
}

// The rows of instructions [0, kSteps) that hold some of a step's n lookups, four
// instructions at a time (the others keep what they held); row id broadcast from lane u of
// this lane's row of 16.  A row id of `rows` (a lookup past n, an invalid id) reads zeros
// through the descriptor, with no access to memory.
template <int S, int U = 0>
__device__ __forceinline__ void issue_rows(const RunInfo& ri, int row, int lane_c, int n, i32x4 (&raw)[kSteps]) {
  if constexpr (U < kSteps) {
    if (U > 0 && U % 4 == 0 && n <= U * S) {
      undefined_rows<U>(raw);
    } else {
      raw[U] = buffer_load_row(ri.rsrc, row_bcast<U>(row), lane_c, 0, 0);
      issue_rows<S, U + 1>(ri, row, lane_c, n, raw);
    }
  }
}
// The same for a table past the descriptor's 32-bit offsets (invalid ids read row 0, their
// values are cleared by clear_rows).
__device__ __forceinline__ void issue_rows_big(const RunInfo& ri, int row, int lane_c, int R, i32x4 (&raw)[kSteps]) {
  GMEM const char* const wb = ri.base() + lane_c;
  static_for<kSteps>([&](auto u) __attribute__((always_inline)) {
    raw[u] = *reinterpret_cast<GMEM const i32x4*>(
        wb + static_cast<uint64_t>(static_cast<uint32_t>(row_bcast<decltype(u)::value>(row))) *
                 static_cast<uint32_t>(R));
  });
}
__device__ __forceinline__ void clear_rows(bool ok, i32x4 (&raw)[kSteps]) {
  const int okv = ok ? 1 : 0;
  static_for<kSteps>([&](auto u) __attribute__((always_inline)) {
    if (!row_bcast<decltype(u)::value>(okv)) raw[u] = zero4();
  });
}

// Lane constants of a walker.
struct LaneConst {
  int lane, sw, lane_sw, lane_c, pos_l;
  bool active, loads, counts;
};

template <int G>
__device__ __forceinline__ LaneConst lane_const(int R) {
  LaneConst l;
  l.lane = threadIdx.x & 63;
  l.sw = l.lane / G;
  l.lane_sw = l.lane & (G - 1);
  l.active = l.lane_sw * 16 < R;
  l.lane_c = l.active ? l.lane_sw * 16 : 0;
  l.pos_l = (l.lane & 15) * (64 / G) + l.sw;   // lookup (or bag) u S + s of instruction u = lane & 15
  l.loads = (l.lane & 15) < kSteps;
  l.counts = l.loads && l.lane_sw < 16;         // one copy of each id is counted
  return l;
}

// ---------------------------------------------------------------- multi-lookup bags

// The bags of a chunk are summed in 32-bit positions relative to `base`, the chunk's first
// lookup (a chunk of more than kFar lookups is rebased on the way), and per instruction of a
// step the scalar unit compares the current bag's end with a constant.  Control is scalar
// throughout -- lanes are masked by selects and dropped stores, and gather.hip is built so
// that uniform branches stay branches -- which leaves a move, a compare and a jump beside
// the additions.  Against 64-bit ends and masked branches (512-byte rows, bags of 20: 7.9
// VALU and 7.5 SALU instructions per lookup, now 4.2 and 4.7): 131M lookups 3751 -> 3605 us,
// 1.9M weighted lookups 86.5 -> 79.7 us; 256-byte fp16 rows in bags of 8, 119.4 -> 108.7 us;
// 384-byte rows in bags of 35, 39.6 -> 33.5 us; 1-KB rows in bags of 3, 34.9 -> 19.7 us.
template <int G, bool F16, bool W>
struct Multi {
  static constexpr int S = 64 / G;
  static constexpr int NA = F16 ? 8 : 4;
  static constexpr int P = NA / S;
  static constexpr int N = S * kSteps;   // lookups per step
  static constexpr int kFar = far_of(N);   // longest stretch of lookups between rebases

  int sw, lane, lane_c, pos_l;
  int loff;                     // this lane's byte offset in a pooled row
  int row_out;                  // bytes of a pooled row
  bool loads, counts;
  int64_t obytes;               // bytes between a bag's pooled row and the next one's

  // the chunk being summed: bags [b, be), lookups [base + q, base + qend)
  RunInfo ri;
  int64_t base, bstart;         // position of q = 0; where bag b starts
  int q, qend, b, be, wb;
  int e;                        // end of bag b, relative to base
  int wrel;                     // lane i: end of bag wb + i, relative to base
  GMEM char* optr;              // bag b's pooled row
  Acc<F16> acc;

  __device__ __forceinline__ void init(const LookupArgs& a) {
    const LaneConst l = lane_const<G>(a.R);
    sw = l.sw;
    lane = l.lane;
    lane_c = l.lane_c;
    pos_l = l.pos_l;
    loff = (NA * l.lane_sw + P * l.sw) * 4;
    row_out = a.E * 4;
    loads = l.loads;
    counts = l.counts;
    obytes = static_cast<int64_t>(a.T) * a.E * 4;
  }

  // ids (and weights) of the n lookups from `first` on, one per lane at pos_l (n > 0; lanes
  // past the end read the last one)
  __device__ __forceinline__ void load_ids(const LookupArgs& a, int64_t first, int n, int64_t& id, float& wt) const {
    const uint32_t x = static_cast<uint32_t>(min(pos_l, n - 1));
    id = *reinterpret_cast<GMEM const int64_t*>(reinterpret_cast<GMEM const char*>(as_global(a.indices) + first) + x * 8u);
    if constexpr (W)
      wt = *reinterpret_cast<GMEM const float*>(reinterpret_cast<GMEM const char*>(as_global(a.weights) + first) + x * 4u);
  }

  __device__ void walk(const LookupArgs& a, const LMEM GatherRun* runs, WaveQueue& qu) {
    const CMEM int64_t* const coff = (const CMEM int64_t*)a.offsets;
    // a chunk's head: where its lookups start and end (scalar loads) and, lane i, where bag
    // bs + i ends (a chunk holds at most 64 bags)
    Chunk nxt;
    int64_t np = 0, npend = 0, nwin = 0;
    auto fetch = [&]() __attribute__((always_inline)) {
      nxt = qu.next();
      if (nxt.run >= 0) {
        const int64_t tb = static_cast<int64_t>(__builtin_amdgcn_readfirstlane(runs[nxt.run].table)) * a.B;
        np = uni64(coff[tb + nxt.bs]);
        npend = uni64(coff[tb + nxt.be]);
        nwin = as_global(a.offsets)[tb + min(nxt.bs + 1 + lane, nxt.be)];
      }
    };
    int64_t pend;
    auto open = [&]() __attribute__((always_inline)) {   // the fetched chunk becomes the current one
      ri = run_info(runs, nxt.run, a);
      base = np;
      pend = npend;
      bstart = np;
      q = 0;
      qend = stretch(npend - np, kFar);
      wb = b = nxt.bs;
      be = nxt.be;
      wrel = rel32(nwin - base);
      e = __builtin_amdgcn_readlane(wrel, 0);
      optr = reinterpret_cast<GMEM char*>(as_global(a.out) + static_cast<int64_t>(ri.table) * a.E) + b * obytes;
    };
    fetch();
    if (nxt.run < 0) return;
    open();
    int64_t id = 0;
    float wt = 0.0f;
    if (qend > 0) load_ids(a, base, min(N, qend), id, wt);
    int ahead = 0;   // 1: the chunk after this one has been looked up (nxt)
    acc_zero(acc);
    while (true) {
      int ids_ready = 0;   // the first ids of the next chunk are in flight
      while (true) {
        if (q >= qend) {
          if (qend < kFar || base + q >= pend) break;
          rebase(a, pend, id, wt);   // (a chunk of more than kFar lookups)
        }
        const int n = uni(min(N, qend - q));
        const bool okp = loads && pos_l < n;
        const bool ok = okp && static_cast<uint64_t>(id) < ri.rows();
        const uint64_t badm = __ballot(okp && !ok && counts);
        float wl = 0.0f;
        if constexpr (W) wl = ok ? wt : 0.0f;
        i32x4 raw[kSteps];
        if (!ri.big()) {
          issue_rows<S>(ri, ok ? static_cast<int>(id) : ri.rsrc.z, lane_c, n, raw);
        } else {
          issue_rows_big(ri, ok ? static_cast<int>(id) : 0, lane_c, a.R, raw);
        }
        // the next chunk's head, two steps before this one ends
        const int left = uni(qend - q - n);
        if (uni(ahead) == 0 && left <= N) {
          fetch();
          ahead = 1;
        }
        // ids of the next step: more of this chunk, or the start of the next one
        if (left > 0) {
          load_ids(a, base + (q + n), min(N, left), id, wt);
        } else if (uni(nxt.run) >= 0 && uni(qend) < kFar && npend > np) {
          load_ids(a, np, min(N, stretch(npend - np, kFar)), id, wt);
          ids_ready = 1;
        }
        asm volatile("" ::: "memory");   // every load of the step is issued before its first use
        if (badm != 0) {   // an out-of-range id is counted and adds nothing
          if (lane == 0) atomicAdd(as_global(a.err), static_cast<unsigned long long>(__popcll(badm)));
        }
        if (ri.big() && __ballot(loads && !ok) != 0) clear_rows(ok, raw);
        consume<0>(a, raw, n, __float_as_int(wl));
        q = uni(q + n);
      }
      // bags left at the chunk's end: one whose last lookup closed the final step (its
      // sum is in acc), then empty ones
      while (uni(b) < uni(be)) {
        finish(q);
        b = uni(b + 1);
      }
      if (uni(ahead) == 0) fetch();
      ahead = 0;
      if (uni(nxt.run) < 0) break;
      open();
      if (uni(ids_ready) == 0 && uni(qend) > 0) load_ids(a, base, min(N, qend), id, wt);
    }
  }

  // moves base to the lookups reached so far, of which more than kFar follow (or followed)
  __device__ __forceinline__ void rebase(const LookupArgs& a, int64_t pend, int64_t& id, float& wt) {
    base = uni64(base + q);
    q = 0;
    qend = uni(stretch(pend - base, kFar));
    wb = b;
    wrel = rel32(as_global(a.offsets)[static_cast<int64_t>(ri.table) * a.B + min(b + 1 + lane, be)] - base);
    e = b < be ? __builtin_amdgcn_readlane(wrel, 0) : INT32_MAX;
    load_ids(a, base, min(N, qend), id, wt);
  }

  // Adds the n lookups of a step: instruction U holds lookups U S + s, one per SW s.  A bag
  // that ends inside an instruction splits its SWs: those before the end add to the ending
  // bag, the others to the next one.  (Lookups past n were loaded as zeros, or not loaded.)
  // Lanes are masked by selects and dropped stores, never by branches: with scalar control
  // alone the compiler keeps one copy of the sums and of the scalar state.
  template <int U>
  __device__ __forceinline__ void consume(const LookupArgs& a, const i32x4 (&raw)[kSteps], int n, int wlb) {
    if constexpr (U < kSteps) {
      if (U > 0 && U % 4 == 0 && n <= U * S) return;
      const float w = W ? __int_as_float(row_bcast<U>(wlb)) : a.one;
      int r = uni(e - q);
      asm volatile("" : "+s"(r));   // one compare per instruction (no chains of jumps between them)
      if (__builtin_expect(r >= (U + 1) * S, 1)) {
        acc_add(acc, raw[U], w);
      } else {
        int lo = 0;
        do {
          const int k = r - U * S;
          if (k > lo) add_only(raw[U], w, sw >= lo && sw < k);
          finish(e);
          b = uni(b + 1);
          lo = k;
          e = uni(b < be ? __builtin_amdgcn_readlane(wrel, b - wb) : INT32_MAX);
          r = uni(e - q);
        } while (r < (U + 1) * S);
        add_only(raw[U], w, sw >= lo);
      }
      consume<U + 1>(a, raw, n, wlb);
    }
  }
  // the lanes' lookups are added where `on` (elsewhere a zero with weight zero: neither an
  // infinity nor a NaN of another bag's row or weight gets in)
  __device__ __forceinline__ void add_only(const i32x4 x, float w, bool on) {
    if constexpr (S == 1) {   // (an end never falls inside an instruction)
      acc_add(acc, x, w);
    } else {
      acc_add(acc, i32x4{on ? x.x : 0, on ? x.y : 0, on ? x.z : 0, on ? x.w : 0}, W ? (on ? w : 0.0f) : w);
    }
  }

  // bag b ends at base + end and is complete in acc: combine the SWs, scale a mean, store, clear
  __device__ __forceinline__ void finish(int end) {
    reduce_scatter<S, NA>(acc.v);
    const int64_t stop = base + end;
    if (ri.mean() && uni64(stop - bstart) > 1) {
      const float s = 1.0f / static_cast<float>(stop - bstart);
#pragma unroll
      for (int i = 0; i < P; ++i) acc.v[i] *= s;
    }
    bstart = uni64(stop);
    const uint64_t o = reinterpret_cast<uint64_t>(optr);
    buffer_store_part<P>(i32x4{static_cast<int>(o), static_cast<int>(o >> 32), row_out, 0x00020000}, loff, acc.v);
    optr = reinterpret_cast<GMEM char*>(uni64(reinterpret_cast<int64_t>(optr) + obytes));
    acc_zero(acc);
  }
};

// ---------------------------------------------------------------- single-lookup bags

template <int G, bool F16, bool W>
__device__ __forceinline__ void single_slow(const LookupArgs& a, const RunInfo& ri, int bs, int be);

template <int G, bool F16, bool W>
struct Single {
  static constexpr int S = 64 / G;
  static constexpr int NA = F16 ? 8 : 4;
  static constexpr int N = S * kSteps;   // bags per step (= per chunk)

  int lane, sw, lane_c, pos_l;
  uint32_t loff;                // byte offset of this lane's piece of its SW's pooled row
  bool active, loads, counts;
  int R;
  int64_t obytes;               // bytes between a bag's pooled row and the next one's

  __device__ __forceinline__ void init(const LookupArgs& a) {
    const LaneConst l = lane_const<G>(a.R);
    lane = l.lane;
    sw = l.sw;
    lane_c = l.lane_c;
    pos_l = l.pos_l;
    active = l.active;
    loads = l.loads;
    counts = l.counts;
    R = a.R;
    obytes = static_cast<int64_t>(a.T) * a.E * 4;
    loff = static_cast<uint32_t>(l.sw) * static_cast<uint32_t>(obytes) + static_cast<uint32_t>(NA * l.lane_sw) * 4u;
  }

  // first and end position of this lane's bag of chunk c (vector loads)
  __device__ __forceinline__ void head(const LookupArgs& a, const RunInfo& ri, const Chunk& c, int64_t& st,
                                       int64_t& en) const {
    GMEM const int64_t* off = as_global(a.offsets) + static_cast<int64_t>(ri.table) * a.B;
    const int bl = min(c.bs + pos_l, c.be);
    st = off[bl];
    en = off[min(bl + 1, c.be)];
  }

  // A three-stage pipeline over chunks: rows of chunk i, ids of chunk i + 1 and the
  // head of chunk i + 2 are in flight together, and each iteration waits once.  Between
  // stages a lane keeps only its bag's masks and id.
  __device__ void walk(const LookupArgs& a, const LMEM GatherRun* runs, WaveQueue& q) {
    Chunk c0 = q.next();
    if (c0.run < 0) return;
    RunInfo r0 = run_info(runs, c0.run, a);
    int64_t st, en;
    head(a, r0, c0, st, en);
    wait_all();
    bool inb0 = loads && c0.bs + pos_l < c0.be;
    bool has0 = inb0 && en > st;
    bool multi0 = inb0 && en - st > 1;
    int64_t id0 = has0 ? as_global(a.indices)[st] : int64_t(-1);
    float w0 = 0.0f;
    if constexpr (W) w0 = has0 ? as_global(a.weights)[st] : 0.0f;
    Chunk c1 = q.next();
    RunInfo r1;
    if (c1.run >= 0) {
      r1 = run_info(runs, c1.run, a);
      head(a, r1, c1, st, en);
    }
    wait_all();
    while (true) {
      // ---- chunk c0: its id has landed; chunk c1's head has landed
      const bool ok = has0 && static_cast<uint64_t>(id0) < r0.rows();
      const uint64_t badm = __ballot(has0 && !ok && counts);
      float wl = 0.0f;
      if constexpr (W) wl = ok ? w0 : 0.0f;
      i32x4 raw[kSteps];
      const int nb = c0.be - c0.bs;
      if (!r0.big())
        issue_rows<S>(r0, ok ? static_cast<int>(id0) : r0.rsrc.z, lane_c, nb, raw);
      else
        issue_rows_big(r0, ok ? static_cast<int>(id0) : 0, lane_c, R, raw);
      bool inb1 = false, has1 = false, multi1 = false;
      int64_t id1 = -1;
      float w1 = 0.0f;
      Chunk c2;
      c2.run = -1;
      RunInfo r2;
      if (c1.run >= 0) {
        inb1 = loads && c1.bs + pos_l < c1.be;
        has1 = inb1 && en > st;
        multi1 = inb1 && en - st > 1;
        id1 = has1 ? as_global(a.indices)[st] : int64_t(-1);
        if constexpr (W) w1 = has1 ? as_global(a.weights)[st] : 0.0f;
        c2 = q.next();
        if (c2.run >= 0) {
          r2 = run_info(runs, c2.run, a);
          head(a, r2, c2, st, en);
        }
      }
      wait_all();   // the one wait of the step
      if (badm != 0 && lane == 0) atomicAdd(as_global(a.err), static_cast<unsigned long long>(__popcll(badm)));
      if (r0.big() && __ballot(loads && !ok) != 0) clear_rows(ok, raw);
      // each SW stores its bag's row (zeros for an empty bag or an out-of-range id)
      GMEM char* const ob = reinterpret_cast<GMEM char*>(as_global(a.out) + static_cast<int64_t>(r0.table) * a.E) +
                            c0.bs * obytes;
      store_rows<0>(a, ob, nb, raw, __float_as_int(wl));
      if (__ballot(multi0) != 0) single_slow<G, F16, W>(a, r0, c0.bs, c0.be);
      if (c1.run < 0) return;
      c0 = c1;
      r0 = r1;
      has0 = has1;
      multi0 = multi1;
      id0 = id1;
      w0 = w1;
      c1 = c2;
      r1 = r2;
    }
  }

  // instruction U's bags U S + s (SW s), those of the chunk's nb
  template <int U>
  __device__ __forceinline__ void store_rows(const LookupArgs& a, GMEM char* ob, int nb, const i32x4 (&raw)[kSteps],
                                             int wlb) const {
    if constexpr (U < kSteps) {
      if (U > 0 && U % 4 == 0 && nb <= U * S) return;
      const float w = W ? __int_as_float(row_bcast<U>(wlb)) : a.one;
      if (U * S + sw < nb && active) store_row(reinterpret_cast<GMEM float*>(ob + loff), raw[U], w);
      store_rows<U + 1>(a, ob + S * obytes, nb, raw, wlb);
    }
  }

  __device__ __forceinline__ void store_row(GMEM float* q, const i32x4 r, float wt) const {
    if constexpr (!W && !F16) {
      const u32x4 v = {static_cast<unsigned>(r.x), static_cast<unsigned>(r.y), static_cast<unsigned>(r.z),
                       static_cast<unsigned>(r.w)};   // fp32 rows are their own output
      __builtin_nontemporal_store(v, reinterpret_cast<GMEM u32x4*>(q));
    } else {
      Acc<F16> x;
      acc_zero(x);
      acc_add(x, r, wt);
      store_part<NA>(q, x.v);
    }
  }
};

// Bags [bs, be) of a single-lookup chunk that hold more than one lookup after all, summed
// again in lookup order, each by the SW that stored its first row (the statistics promised
// at most one lookup per bag).  Rare: the offsets are read again.
template <int G, bool F16, bool W>
__device__ __forceinline__ void single_slow(const LookupArgs& a, const RunInfo& ri, int bs, int be) {
  constexpr int S = 64 / G;
  constexpr int NA = F16 ? 8 : 4;
  const LaneConst l = lane_const<G>(a.R);
  const int64_t ostride = static_cast<int64_t>(a.T) * a.E;
  GMEM const int64_t* off = as_global(a.offsets) + static_cast<int64_t>(ri.table) * a.B;
  GMEM const int64_t* indices = as_global(a.indices);
  GMEM const float* wts = as_global(a.weights);
  for (int u = 0; u < kSteps; ++u) {
    const int bi = u * S + l.sw;
    if (bs + bi < be) {
      const int64_t st = off[bs + bi], en = off[bs + bi + 1];
      if (en - st > 1) {
        Acc<F16> acc;
        acc_zero(acc);
        for (int64_t k = st; k < en; ++k) {
          const int64_t x = indices[k];
          const bool ok = static_cast<uint64_t>(x) < ri.rows();
          if (!ok && k > st && l.lane_sw == 0) atomicAdd(as_global(a.err), 1ull);   // the first id was counted
          const float wk = W ? (ok ? wts[k] : 0.0f) : a.one;
          i32x4 r = load_row(ri, ok ? static_cast<int>(x) : 0, l.lane_c, a.R);
          if (!ok) r = zero4();
          acc_add(acc, r, wk);
        }
        if (ri.mean()) {
          const float sc = 1.0f / static_cast<float>(en - st);
#pragma unroll
          for (int i = 0; i < NA; ++i) acc.v[i] *= sc;
        }
        if (l.active)
          store_part<NA>(as_global(a.out) + static_cast<int64_t>(ri.table) * a.E + static_cast<int64_t>(bs + bi) * ostride +
                             NA * l.lane_sw,
                         acc.v);
      }
    }
  }
}

#ifdef EMBX_WAVES_PER_EU
#define EMBX_OCCUPANCY __attribute__((amdgpu_waves_per_eu(EMBX_WAVES_PER_EU, EMBX_WAVES_PER_EU)))
#else
#define EMBX_OCCUPANCY
#endif

// W: every lookup carries a weight (a.weights).
template <int G, bool F16, bool W>
__global__ void __launch_bounds__(kBlock) EMBX_OCCUPANCY gather_kernel(LookupArgs a) {
  extern __shared__ __align__(16) char smem_raw[];
  __shared__ int s_ctr[2];
  LMEM char* lds = (LMEM char*)smem_raw;
  const int wg = blockIdx.x;
  const int tid = threadIdx.x;
  GMEM unsigned long long* tw =
      a.trace ? as_global(a.trace) + static_cast<int64_t>(wg) * kTraceWorker : nullptr;
  if (tw && tid == 0) tw[0] = __builtin_amdgcn_s_memrealtime();
  {   // the worker's slot: a header record, then its runs
    GMEM const char* src = reinterpret_cast<GMEM const char*>(as_global(a.gr) + static_cast<int64_t>(wg) * a.gr_slot);
    for (int q = tid; q < 3 * a.gr_slot; q += kBlock) {
      uint4 x = *reinterpret_cast<GMEM const uint4*>(src + 16 * q);
      if (q >= 3 && q % 3 == 1) {   // (table, j, k, cb) of a run: slice j of k as bags [floor(jB / k), floor((j+1)B / k))
        const double B = a.B, j = static_cast<double>(x.y), k = static_cast<double>(x.z);
        // exact: j B < 2^47, and a quotient below an integer is below it by 1/k >= 2^-16, far
        // more than the division's rounding
        x.y = static_cast<uint32_t>(j * B / k);
        x.z = static_cast<uint32_t>((j + 1.0) * B / k);
      }
      *reinterpret_cast<LMEM uint4*>(lds + 16 * q) = x;
    }
  }
  constexpr int waves = kBlock >> 6;   // (a compile-time count: read from blockDim it costs ~35 VGPRs)
  if (tid == 0) {
    s_ctr[0] = waves;
    s_ctr[1] = waves;
  }
  if (tw && tid == 0) tw[1] = __builtin_amdgcn_s_memrealtime();
  __syncthreads();
  const LMEM GatherSlotHeader* hd = reinterpret_cast<const LMEM GatherSlotHeader*>(lds);
  const int n_single = __builtin_amdgcn_readfirstlane(hd->n_single);
  const int single_chunks = __builtin_amdgcn_readfirstlane(hd->single_chunks);
  const int multi_chunks = __builtin_amdgcn_readfirstlane(hd->sw_chunks);
  const int nr = __builtin_amdgcn_readfirstlane(hd->n_runs);
  const LMEM GatherRun* runs = reinterpret_cast<const LMEM GatherRun*>(lds + sizeof(GatherRun));
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  if (n_single > 0) {
    WaveQueue q{runs, 0, n_single, single_chunks, (LMEM int*)&s_ctr[0], wave, waves};
    Single<G, F16, W> w;
    w.init(a);
    w.walk(a, runs, q);
  }
  if (nr > n_single) {
    // the wavefronts that took a single-lookup chunk take their first multi-lookup chunk
    // last, so that the others start on this queue at once (a permutation of [0, waves):
    // every chunk below `waves` is still some wavefront's first)
    const int busy = n_single > 0 ? min(single_chunks, waves) : 0;
    WaveQueue q{runs, n_single, nr, multi_chunks, (LMEM int*)&s_ctr[1], (wave + waves - busy) % waves, waves};
    Multi<G, F16, W> w;
    w.init(a);
    w.walk(a, runs, q);
  }
  if (tw && (tid & 63) == 0) tw[2 + (tid >> 6)] = __builtin_amdgcn_s_memrealtime();
}

using GatherFn = void (*)(LookupArgs);

template <bool F16, bool W>
GatherFn pick_gather(int G) {
  switch (G) {
    case 16: return &gather_kernel<16, F16, W>;
    case 32: return &gather_kernel<32, F16, W>;
    case 64: return &gather_kernel<64, F16, W>;
    default: return nullptr;
  }
}

}  // namespace

#define EMBX_GNAME2(name, ks) name##_k##ks
#define EMBX_GNAME(name, ks) EMBX_GNAME2(name, ks)
#if EMBX_HAS_GPART(0)
GatherKernelFn EMBX_GNAME(gather_kernel_f32, EMBX_GKS)(int G) { return pick_gather<false, false>(G); }
#endif
#if EMBX_HAS_GPART(1)
GatherKernelFn EMBX_GNAME(gather_kernel_f32_weighted, EMBX_GKS)(int G) { return pick_gather<false, true>(G); }
#endif
#if EMBX_HAS_GPART(2)
GatherKernelFn EMBX_GNAME(gather_kernel_f16, EMBX_GKS)(int G) { return pick_gather<true, false>(G); }
#endif
#if EMBX_HAS_GPART(3)
GatherKernelFn EMBX_GNAME(gather_kernel_f16_weighted, EMBX_GKS)(int G) { return pick_gather<true, true>(G); }
#endif

}  // namespace embx
