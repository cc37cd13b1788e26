// Fused local update + P-Reduce for CDNA4 (gfx950).
//
// One launch runs one step of the algorithm of Fig. 4 for every scheduled
// unit of work: a group G (Step 4, the F^G of Sec. 3.2, with the Step 2
// update of its members that compute this step folded in) or a worker that
// updates without synchronizing.  Disjoint groups run concurrently (Sec. 3.2).
//
// Work decomposition.  Every unit touches the same element range of its
// members' buffers, so the launch is a list of (unit, tile) work items, one
// per single-wave workgroup, unit after unit.  A tile is 64 lanes x 1-4
// slots x 16 bytes of each member stream; the slot count shrinks as the
// unit's number of streams grows (see slot_log2), so every lane keeps 8-16
// 16-byte loads in flight (24 for a group of eight with momentum).  The host
// caps residency per launch at 4-14 waves per CU (an LDS reservation; 16 where
// that many hold the whole launch), fewer when the units read more streams:
// HBM3E delivered its best rate at a bounded depth of outstanding requests, not
// at full occupancy.  Groups above eight
// have a kernel of their own (wide_step_kernel).
// A workgroup handles one unit, so the unit's size k, its member ids and their active
// flags are wave-uniform: they sit in scalar registers and every branch on
// them is a scalar branch.  Each thread issues the loads of all members
// (and their gradients / momenta) for all its slots before any arithmetic,
// then writes the mean back to every member.
//
// The operation is a stream over HBM with no data reuse and about one flop
// per 4 bytes, so there is no LDS tiling and no matrix-core work: the design
// aims at full-width (dwordx4) coalesced accesses and enough bytes in flight
// per CU.
//
// Arithmetic follows the exact fp32 order documented in include/rip.h (no
// contraction into FMA, sequential sum in ascending member order, product
// with (float)(1.0/k)); bf16 values widen exactly and round to nearest-even
// once when stored.

#include <hip/hip_runtime.h>

#include <cstdint>

#include "rip_kernel_args.h"

#pragma clang fp contract(off)

namespace rip {
namespace {

typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));

// Tiles are accessed through buffer instructions, non-temporal (every
// byte is touched once per step): a descriptor per member stream whose base
// is the tile's first byte and whose size is the tile's bytes, and a
// per-lane offset of at most a few KB.  On gfx950 this form streamed 3-4%
// faster than the same non-temporal accesses as global instructions (with a
// 64-bit per-lane address or an SGPR base and 32-bit offset alike), and
// faster than a buffer descriptor over the whole stream with the tile offset
// folded into the per-lane offset.  The descriptor's size also bounds every
// access in hardware.
typedef __amdgpu_buffer_rsrc_t Rsrc;
constexpr int kRsrcWord3 = 0x00020000;  // raw (untyped) buffer, 32-bit data format
constexpr int kNonTemporal = 2;         // cache-policy operand: nt

__device__ __forceinline__ Rsrc tile_rsrc(const char* tile, int bytes) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<char*>(tile), 0, bytes, kRsrcWord3);
}
__device__ __forceinline__ u32x4 bld16(Rsrc r, int off) {
  return __builtin_amdgcn_raw_buffer_load_b128(r, off, 0, kNonTemporal);
}
__device__ __forceinline__ void bst16(Rsrc r, int off, u32x4 v) {
  __builtin_amdgcn_raw_buffer_store_b128(v, r, off, 0, kNonTemporal);
}

// The launch tables -- the kernel argument's own arrays (unit tables, member
// ids, active bits) and the registered pointer and segment tables -- are
// never written while a launch runs.  Reading them through the constant
// address space lets the compiler fetch these wave-uniform values with
// scalar loads, also inside divergent code; read as ordinary global memory
// they become vector loads that wait behind the streaming traffic (the
// kernel's own stores could alias them, as far as the compiler can tell).
// The argument's arrays are read where the argument lives, in the kernel-
// argument segment (the only explicit argument, at its start), never through
// the address of a by-value copy, which is private memory in an unoptimized
// build.
#define RIP_CONST __attribute__((address_space(4)))

typedef const RIP_CONST StepArgs KArgs;
__device__ __forceinline__ KArgs& kargs() {
  return *(KArgs*)__builtin_amdgcn_kernarg_segment_ptr();
}

template <typename T>
__device__ __forceinline__ T cld(const T* p, int64_t i) {
  return ((const RIP_CONST T*)p)[i];
}
template <typename T>
__device__ __forceinline__ T cld(const RIP_CONST T* p, int64_t i) {
  return p[i];
}
// Bytes i .. i+7 of the (16-byte aligned, padded) member table as one 64-bit
// value, byte j in bits 8j..8j+7: one 16-byte scalar load of the aligned
// dwords that hold them, then a funnel shift.
typedef uint32_t u32x4c __attribute__((ext_vector_type(4)));
__device__ __forceinline__ uint64_t cld8x8(const RIP_CONST uint8_t* p, int i) {
  const u32x4c d = ((const RIP_CONST u32x4c*)p)[i >> 4];
  const u32x4c e = ((const RIP_CONST u32x4c*)p)[(i >> 4) + 1];
  // 32 bytes d|e hold bytes (i & ~15) .. (i & ~15) + 31, which cover i .. i+7
  const int sh = (i & 15) * 8;  // 0..120
  const uint64_t q0 = d.x | ((uint64_t)d.y << 32), q1 = d.z | ((uint64_t)d.w << 32);
  const uint64_t q2 = e.x | ((uint64_t)e.y << 32);
  if (sh == 0) return q0;
  if (sh < 64) return (q0 >> sh) | (q1 << (64 - sh));
  if (sh == 64) return q1;
  return (q1 >> (sh - 64)) | (q2 << (128 - sh));
}

__device__ __forceinline__ float bf16_lo(uint32_t x) { return __uint_as_float(x << 16); }
__device__ __forceinline__ float bf16_hi(uint32_t x) { return __uint_as_float(x & 0xFFFF0000u); }

// fp32 -> bf16, round to nearest even, NaN kept quiet: gfx950's
// v_cvt_pk_bf16_f32 (what clang emits for a conversion to __bf16), two values
// per instruction.  Its results equal the round-to-nearest-even definition
// for all 2^32 fp32 inputs (tests/test_gpu_ieee_edges.py runs every one).
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));

__device__ __forceinline__ uint32_t bf16_pack2(float lo, float hi) {
  const f32x2 f = {lo, hi};
  return __builtin_bit_cast(uint32_t, __builtin_convertvector(f, bf16x2));
}
template <bool BF16>
struct Vec;

// 16 bytes = 4 fp32
template <>
struct Vec<false> {
  static constexpr int N = 4;
  static __device__ __forceinline__ void unpack(u32x4 x, float (&f)[N]) {
    f[0] = __uint_as_float(x.x);
    f[1] = __uint_as_float(x.y);
    f[2] = __uint_as_float(x.z);
    f[3] = __uint_as_float(x.w);
  }
  static __device__ __forceinline__ u32x4 pack(const float (&f)[N]) {
    u32x4 x;
    x.x = __float_as_uint(f[0]);
    x.y = __float_as_uint(f[1]);
    x.z = __float_as_uint(f[2]);
    x.w = __float_as_uint(f[3]);
    return x;
  }
};

// 16 bytes = 8 bf16; element 2i is the low half of word i
template <>
struct Vec<true> {
  static constexpr int N = 8;
  static __device__ __forceinline__ void unpack(u32x4 x, float (&f)[N]) {
    f[0] = bf16_lo(x.x); f[1] = bf16_hi(x.x);
    f[2] = bf16_lo(x.y); f[3] = bf16_hi(x.y);
    f[4] = bf16_lo(x.z); f[5] = bf16_hi(x.z);
    f[6] = bf16_lo(x.w); f[7] = bf16_hi(x.w);
  }
  static __device__ __forceinline__ u32x4 pack(const float (&f)[N]) {
    u32x4 x;
    x.x = bf16_pack2(f[0], f[1]);
    x.y = bf16_pack2(f[2], f[3]);
    x.z = bf16_pack2(f[4], f[5]);
    x.w = bf16_pack2(f[6], f[7]);
    return x;
  }
};

// (float)(1.0/k) for every group size, evaluated at compile time.
struct InvTable {
  float v[RIP_MAX_REPLICAS + 1];
};
constexpr InvTable make_inv_table() {
  InvTable t{};
  for (int k = 1; k <= RIP_MAX_REPLICAS; ++k) t.v[k] = (float)(1.0 / k);
  return t;
}
__constant__ InvTable kInv = make_inv_table();

// Step 2 for one element (fp32, this order, no contraction):
//   g' = g + wd*w                       (only when weight decay is on)
//   SGD:       u = w - lr*g'
//   momentum:  v = mu*v + g';  u = w - lr*v,  or with Nesterov u = w - lr*(g' + mu*v)
// EXT selects the kernel variant that handles weight decay and Nesterov.
// Their flags are wave-uniform, but the compiler turns the tests into
// per-element selects, computing both sides: that more than doubles the
// arithmetic per element, which costs bandwidth when few waves share a CU.
// Plain SGD and heavy-ball momentum therefore get a variant without them;
// with wd == 0 and no Nesterov both variants compute the same values.
struct Opt {
  float lr, mu, wd;
  bool nesterov;
};

template <bool MOM, bool EXT>
__device__ __forceinline__ float update(float w, float g, float& v, const Opt& o) {
  if constexpr (EXT) {
    if (o.wd != 0.0f) g = g + o.wd * w;
  }
  if constexpr (MOM) {
    v = o.mu * v + g;
    if constexpr (EXT) return w - o.lr * (o.nesterov ? g + o.mu * v : v);
    return w - o.lr * v;
  } else {
    return w - o.lr * g;
  }
}

// Launch-wide values, read once per work item before anything else.
struct Header {
  const RIP_CONST uint64_t* ptab;
  const RIP_CONST int64_t *seg_numel, *seg_tile0;
  uint32_t work, blocks, uniform_k;
  int n_seg, n_rep, n_units, one_slot;
  int64_t flat_numel;
  Opt opt;
};

__device__ __forceinline__ int lane_id() { return (int)threadIdx.x & (kBlock - 1); }

// The last element of a bf16 tile of odd size is the low half of a dword.  The
// loads take that dword whole: an aligned dword lies in one page, so what
// follows the element can be read, and it is never stored.  The stores leave
// the dword out and store the element alone, from slot e / 64 of lane e % 64,
// e its vector.  (Loaded alone too, it cost the ragged waves another round of
// loads and code of their own: 8 lone bf16 replicas of 2,007 2.19 us a launch,
// now 1.95; one group of 256 of 65,539 31.7, now 25.6.)
__device__ __forceinline__ int load_bytes(int bytes) { return (bytes + 3) & ~3; }
constexpr int kOutside = 0x7FFFFFF0;  // a byte offset past every tile

template <int U, typename F>
__device__ __forceinline__ void odd_store(char* tile, int bytes, F&& vec) {
  const int at = bytes - 2, e = at >> 4, word = (at >> 2) & 3;
  const int off = (e & (kBlock - 1)) == lane_id() ? at : kOutside;
  uint32_t x = 0;
#pragma unroll
  for (int u = 0; u < U; ++u)
#pragma unroll
    for (int i = 0; i < 4; ++i) x = (u == e / kBlock && i == word) ? vec(u)[i] : x;
  __builtin_amdgcn_raw_buffer_store_b16((uint16_t)x, tile_rsrc(tile, bytes), off, 0, kNonTemporal);
}

struct Members {
  char* w[kMaxK];
  const char* g[kMaxK];
  char* v[kMaxK];
  uint32_t act;  // update flags, bit j = member j
  __device__ __forceinline__ bool active(int j) const {
    return __builtin_expect((act >> j) & 1u, 1);
  }
};

// The unit's member ids (one per byte of `ids`) came with the unit; their
// table entries are independent scalar loads, all issued before one wait.
template <int K, bool MOM>
__device__ __forceinline__ void load_members(const Header& h, uint64_t ids, uint32_t act8,
                                             int seg, Members& m) {
#pragma unroll
  for (int j = 0; j < K; ++j) {
    const int id = (int)((ids >> (8 * j)) & 0xFFu);
    const RIP_CONST uint64_t* e = h.ptab + (uint32_t)(seg * h.n_rep + id) * 3u;
    m.w[j] = reinterpret_cast<char*>(e[0]);
    m.g[j] = reinterpret_cast<const char*>(e[1]);
    if constexpr (MOM) m.v[j] = reinterpret_cast<char*>(e[2]);
  }
  m.act = act8;
  // Materialize every member's pointers and flag here, so one wait covers
  // all of these scalar loads.  Left alone, the compiler sinks each pointer
  // load next to its use, and every vector load then waits for its own
  // scalar round trip: the wave's loads go out one at a time.
#pragma unroll
  for (int j = 0; j < K; ++j) {
    asm volatile("" ::"s"(m.w[j]), "s"(m.g[j]));
    if constexpr (MOM) asm volatile("" ::"s"(m.v[j]));
  }
}

// Up to U consecutive 16-byte slots of a tile for a unit of K members; the
// tile starts `tile_byte` bytes into every member stream and holds `bytes`
// (the last tile of a segment: what is left of it).
//
// A ragged end needs no code of its own: the descriptors end at the last
// dword, and the hardware checks each dword of an access against that (a dword
// beyond loads as 0 and is not stored).  Only a bf16 segment of odd size has
// an element in half a dword, which the lane of its vector stores by itself.  (Element by element, each member's loads after the last
// one's, a ragged tile held its wave for tens of microseconds: 16 fp32
// replicas of 304,327 with momentum, weight decay and groups of four 20.5 us
// a step, now 19.1, and 18.4 with a size that ends on a tile; the same as 59
// separate tensors 21.7, now 20.0.)
template <int K, int U, bool BF16, bool MOM, bool EXT, bool PACE>
__device__ __forceinline__ void tile_slots(Members& m, int64_t tile_byte, int bytes,
                                           const Opt& o) {
  using V = Vec<BF16>;
  constexpr int N = V::N;
  constexpr float inv_k = (float)(1.0 / K);
  int off[U];  // this lane's byte offset of each slot within the tile
#pragma unroll
  for (int u = 0; u < U; ++u) off[u] = (u * kBlock + (int)threadIdx.x) * 16;
#pragma unroll
  for (int j = 0; j < K; ++j) {
    m.w[j] += tile_byte;
    m.g[j] += tile_byte;
    if constexpr (MOM) m.v[j] += tile_byte;
  }
  const bool odd = BF16 && (bytes & 2);
  u32x4 wv[U][K], gv[U][K], vv[U][K];
#pragma unroll
  for (int u = 0; u < U; ++u)
#pragma unroll
    for (int j = 0; j < K; ++j) {
      wv[u][j] = bld16(tile_rsrc(m.w[j], load_bytes(bytes)), off[u]);
      if (m.active(j)) {
        gv[u][j] = bld16(tile_rsrc(m.g[j], load_bytes(bytes)), off[u]);
        if constexpr (MOM) vv[u][j] = bld16(tile_rsrc(m.v[j], load_bytes(bytes)), off[u]);
      }
    }
  // From here on the flags and the descriptors' size are new values to the
  // compiler: a descriptor (four scalar registers) lives for its loads only
  // and is put together again for its stores, and a flag is tested where it
  // is used.  Kept over the whole function, up to 24 descriptors and as many
  // branch masks overflowed the scalar registers into VGPR lanes.
  asm volatile("" : "+s"(m.act), "+s"(bytes));
  // All arithmetic comes before the first store.  Stores count against the
  // same vmcnt as loads, and because the gradient and momentum loads are
  // conditional (active members only) the compiler's waits before each
  // member's arithmetic are conservative: a momentum store issued between two
  // members would make the next wait cover that store's completion, a full
  // write round trip.  (A straight-line variant for groups whose members all
  // update, with exact waits, measured no faster and slowed bf16 by 2%.)
  u32x4 out[U];
#pragma unroll
  for (int u = 0; u < U; ++u) {
    float s[N];
#pragma unroll
    for (int j = 0; j < K; ++j) {
      float x[N];
      V::unpack(wv[u][j], x);
      if (m.active(j)) {
        float g[N], v[N];
        V::unpack(gv[u][j], g);
        if constexpr (MOM) V::unpack(vv[u][j], v);
#pragma unroll
        for (int i = 0; i < N; ++i) x[i] = update<MOM, EXT>(x[i], g[i], v[i], o);
        if constexpr (MOM) vv[u][j] = V::pack(v);
      }
#pragma unroll
      for (int i = 0; i < N; ++i) s[i] = (j == 0) ? x[i] : s[i] + x[i];
    }
    if constexpr (K > 1) {
#pragma unroll
      for (int i = 0; i < N; ++i) s[i] = s[i] * inv_k;
    }
    out[u] = V::pack(s);
  }
  // Keep the instruction scheduler from sinking arithmetic below the stores.
  __builtin_amdgcn_sched_barrier(0);
  asm volatile("" : "+s"(m.act));
  // A wave of a large group with momentum has 12-16 stores, and issued back
  // to back they cost the HBM3E rate: 16 cycles between them gave groups of
  // six to eight of 25.6M to 276M elements 0.3-1.5% (eight of 138.4M fp32
  // 7546 -> 7475 us); with fewer streams the pause itself costs (groups of
  // eight without momentum -2%, lone updates with it -2%).
  const auto pace = [] {
    if constexpr (PACE) {
      __builtin_amdgcn_sched_barrier(0);
      asm volatile("s_nop 15");
      __builtin_amdgcn_sched_barrier(0);
    }
  };
  if constexpr (MOM) {
#pragma unroll
    for (int u = 0; u < U; ++u)
#pragma unroll
      for (int j = 0; j < K; ++j) {
        if (m.active(j)) bst16(tile_rsrc(m.v[j], bytes & ~3), off[u], vv[u][j]);
        pace();
      }
  }
#pragma unroll
  for (int u = 0; u < U; ++u)
#pragma unroll
    for (int j = 0; j < K; ++j) {
      bst16(tile_rsrc(m.w[j], bytes & ~3), off[u], out[u]);
      pace();
    }
  if constexpr (BF16) {
    if (__builtin_expect(odd, 0)) {
#pragma unroll
      for (int j = 0; j < K; ++j) {
        if constexpr (MOM)
          if (m.active(j)) odd_store<U>(m.v[j], bytes, [&](int u) { return vv[u][j]; });
        odd_store<U>(m.w[j], bytes, [&](int u) { return out[u]; });
      }
    }
  }
}

// Last index i in [0, n) with v[i] <= x (v ascending, v[0] <= x).
template <typename P, typename X>
__device__ __forceinline__ int last_le(P v, int n, X x) {
  int lo = 0, hi = n - 1;
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    if ((X)cld(v, mid) <= x) lo = mid; else hi = mid - 1;
  }
  return lo;
}

// The unit a workgroup works on, as the main loop decoded it.
struct Unit {
  int base, k;    // member[base .. base + k)
  uint32_t act8;  // update flags of members 0..7
  uint64_t ids;   // member ids 0..7, one per byte
};

__device__ __forceinline__ Header load_header(KArgs* a) {
  // Load the whole header into scalar registers in one batch up front: left
  // to itself the compiler spreads it over several batches (and loads
  // flat_numel late, through a select of addresses), and every extra batch is
  // one more dependent scalar round trip before the workgroup's first vector
  // load.
  const Header h{(const RIP_CONST uint64_t*)a->ptab, (const RIP_CONST int64_t*)a->seg_numel,
                 (const RIP_CONST int64_t*)a->seg_tile0, a->work, a->blocks, a->uniform_k, a->n_seg,
                 a->n_rep, a->n_units, a->one_slot, a->flat_numel,
                 Opt{a->lr, a->mu, a->wd, a->nesterov != 0}};
  asm volatile("" ::"s"(h.ptab), "s"(h.seg_numel), "s"(h.seg_tile0), "s"(h.work), "s"(h.blocks), "s"(h.uniform_k), "s"(h.n_seg),
               "s"(h.n_rep), "s"(h.n_units), "s"(h.one_slot), "s"(h.flat_numel), "s"(h.opt.lr), "s"(h.opt.mu),
               "s"(h.opt.wd), "s"((int)h.opt.nesterov));
  return h;
}

// The unit and tile of work item w.  A launch of units with the same tile
// count has a grid of one row per unit; otherwise the grid is one row of work
// items, unit after unit.
__device__ __forceinline__ int find_unit(KArgs* a, const Header& h, uint32_t w, int64_t& tile) {
  if (h.blocks == 0) {
    tile = (int64_t)w;
    return (int)blockIdx.y;
  }
  const int unit = last_le(a->unit_work0, h.n_units, w);
  tile = (int64_t)(w - cld(a->unit_work0, unit));
  return unit;
}

// Where a tile lies: its segment, first element and element count.
struct Place {
  int seg, elems;
  int64_t e_tile;
};

// The place of tile `tile` of a unit, for tiles of TE elements (slot option
// O).  A flat handle needs no search.
template <int64_t TE>
__device__ __forceinline__ Place find_place(const Header& h, int O, int64_t tile) {
  Place p;
  int64_t numel;
  if (h.n_seg == 1) {
    p.seg = 0;
    p.e_tile = tile * TE;
    numel = h.flat_numel;
  } else {
    const RIP_CONST int64_t* tile0 = h.seg_tile0 + O * (h.n_seg + 1);
    p.seg = last_le(tile0, h.n_seg, tile);
    p.e_tile = (tile - cld(tile0, p.seg)) * TE;
    numel = cld(h.seg_numel, p.seg);
  }
  p.elems = (int)(p.e_tile + TE <= numel ? TE : numel - p.e_tile);
  return p;
}

// One tile of a unit of K members.  The tile geometry is a compile-time constant here, so a
// workgroup reaches its first vector load after a handful of scalar
// instructions: a flat handle needs no segment search at all.
template <int K, int O, bool BF16, bool MOM, bool EXT, bool PACE>
__device__ __forceinline__ void tile_of(const Header& h, const Unit& u, int64_t tile) {
  constexpr int SL = 1 << O;
  constexpr int N = Vec<BF16>::N;
  constexpr int64_t TE = (int64_t)kBlock * N * SL;  // elements per tile
  const Place at = find_place<TE>(h, O, tile);
  constexpr int esize = BF16 ? 2 : 4;
  Members m;
  load_members<K, MOM>(h, u.ids, u.act8, at.seg, m);
  tile_slots<K, SL, BF16, MOM, EXT, PACE>(m, at.e_tile * esize, at.elems * esize, h.opt);
}
// A launch small enough for one-slot tiles leaves HBM idle, and the pause
// between the stores of large momentum groups only costs there: up to 512 tiles
// 5-10%, at 1024 nothing (two groups of eight of 16,384: 3.40 us with it, 3.20
// without; bf16 3.89 and 3.57).  Such a launch has code of its own (3.27 us,
// bf16 3.57); a branch over each pause took back half of it for bf16.
template <int K, bool BF16, bool MOM, bool EXT>
__device__ __forceinline__ void unit_tile(const Header& h, const Unit& u, int64_t tile) {
  constexpr int O = slot_log2(K, MOM);
  constexpr bool kPace = MOM && K >= 6;
  if constexpr (O > 0 || kPace) {
    if (h.one_slot) {
      tile_of<K, 0, BF16, MOM, EXT, false>(h, u, tile);
      return;
    }
  }
  tile_of<K, O, BF16, MOM, EXT, kPace>(h, u, tile);
}

template <bool BF16, bool MOM, bool EXT>
__global__ __launch_bounds__(kBlock) void fused_step_kernel(StepArgs) {
  uint32_t w = blockIdx.x;
  for (;;) {
    // The argument's address is hidden from the optimizer anew for every work
    // item, so nothing is computed ahead of the loop.  A workgroup almost
    // always runs one item (it loops only above the workgroup limit), and
    // values hoisted for all sizes of unit, most of them spilled to VGPR
    // lanes, delayed every wave's first load (two replicas of 16,384: 2.27 us
    // a launch, now 1.93, of which an empty kernel takes 1.65).
    KArgs* a = &kargs();
    asm volatile("" : "+s"(a));
    const Header h = load_header(a);
    int64_t tile;
    const int unit = find_unit(a, h, w, tile);
    // With equal-sized units the member window's address needs no load, so
    // it is fetched together with the unit's info word: the unit costs one
    // scalar round trip, its members' pointers a second.
    const uint32_t info = cld(a->unit_info, unit);
    Unit u;
    if (h.uniform_k) {
      u.k = (int)h.uniform_k;
      u.base = unit * u.k;
    } else {
      u.k = (int)unit_info_k(info);
      u.base = (int)unit_info_base(info);
    }
    u.act8 = unit_info_act8(info);
    u.ids = cld8x8(a->member, u.base);
    switch (u.k) {
      case 1: unit_tile<1, BF16, MOM, EXT>(h, u, tile); break;
      case 2: unit_tile<2, BF16, MOM, EXT>(h, u, tile); break;
      case 3: unit_tile<3, BF16, MOM, EXT>(h, u, tile); break;
      case 4: unit_tile<4, BF16, MOM, EXT>(h, u, tile); break;
      case 5: unit_tile<5, BF16, MOM, EXT>(h, u, tile); break;
      case 6: unit_tile<6, BF16, MOM, EXT>(h, u, tile); break;
      case 7: unit_tile<7, BF16, MOM, EXT>(h, u, tile); break;
      default: unit_tile<8, BF16, MOM, EXT>(h, u, tile); break;
    }
    if (h.blocks == 0) return;
    w += h.blocks;
    if (w >= h.work) return;
  }
}

// Groups larger than kMaxK (All-Reduce as one group of every worker, large
// divisions): one workgroup per tile (one 16-byte slot per lane), its waves
// sharing the members.  A wave holds c <= kWideC members, issues all their
// loads together and updates them; the sum then passes from wave to wave
// through LDS, so it is still taken in ascending member order, and the wave
// with the last members hands the mean to all.  A group of more members than
// the waves hold goes in rounds; a wave loads its next members while the sum
// is with the others.
//
// Bound by the latency of a workgroup where a launch is small, and by the
// number of streams open at once where it is large.  Single waves that took
// the members in chunks of eight one after the other waited for every chunk's
// loads by themselves and left most of the chip idle on small replicas: 256
// bf16 replicas of 65,539 93.2 us, now 25.6; 64 fp32 of 10,000 21.8, now 7.0;
// 9 fp32 of 4M 85.1, now 70.2; 32 fp32 of 25.6M 1797, now 1750 (5.6 TB/s).
// Launches of more than 256 workgroups per CU are 1-7% ahead of them, momentum
// groups above 64 level; pitches of a power of two up to 20% behind.  Four
// members a wave: with eight, the updated values of a bf16 wave take 150-185
// VGPRs, and one workgroup fits a CU (64 bf16 of 2.5M 221 us, now 176); two or
// four slots per lane helped only at one size in ten.
//
// Each turn waits for the one before it only, on a counter in LDS that the
// wave holding the sum advances; every turn belongs to a wave of the same
// workgroup, which takes its turns in ascending order, so every wait ends.
constexpr uint32_t kWideDone = ~0u;  // the turn counter once the mean is there
struct WideShared {
  float sum[8][kBlock];  // [element of the lane's vector][lane]
  u32x4 mean[kBlock];
  uint32_t turn;
};

__device__ __forceinline__ void wait_turn(uint32_t* turn, uint32_t t) {
  while ((uint32_t)__builtin_amdgcn_readfirstlane(
             (int)__hip_atomic_load(turn, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP)) != t) {
  }
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}
__device__ __forceinline__ void pass_turn(uint32_t* turn, uint32_t t) {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
  __hip_atomic_store(turn, t, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}

// Pointers of the members at base .. base + kWideC - 1 of the member table, to
// the tile (all of them, or only the parameters; the table's entries past the
// unit belong to the next one or are 0, and are not used).
template <bool ALL, bool MOM>
__device__ __forceinline__ void wide_members(KArgs* a, const Header& h, int base, int seg,
                                             int64_t tile_byte, Members& m) {
  const uint64_t ids = cld8x8(a->member, base);
#pragma unroll
  for (int j = 0; j < kWideC; ++j) {
    const int id = (int)((ids >> (8 * j)) & 0xFFu);
    const RIP_CONST uint64_t* e = h.ptab + (uint32_t)(seg * h.n_rep + id) * 3u;
    m.w[j] = reinterpret_cast<char*>(e[0]) + tile_byte;
    if constexpr (ALL) {
      m.g[j] = reinterpret_cast<const char*>(e[1]) + tile_byte;
      if constexpr (MOM) m.v[j] = reinterpret_cast<char*>(e[2]) + tile_byte;
    }
  }
#pragma unroll
  for (int j = 0; j < kWideC; ++j) {
    asm volatile("" ::"s"(m.w[j]));
    if constexpr (ALL) {
      asm volatile("" ::"s"(m.g[j]));
      if constexpr (MOM) asm volatile("" ::"s"(m.v[j]));
    }
  }
}

template <bool BF16, bool MOM, bool EXT>
__global__ __launch_bounds__(kBlock * kWideWaves) void wide_step_kernel(StepArgs) {
  using V = Vec<BF16>;
  constexpr int N = V::N;
  constexpr int64_t TE = (int64_t)kBlock * N;
  constexpr int esize = BF16 ? 2 : 4;
  __shared__ WideShared sh;
  const int lane = lane_id();
  const int off = lane * 16;
  const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x / kBlock);
  uint32_t w = blockIdx.x;
  for (;;) {
    if (threadIdx.x == 0) sh.turn = 0;
    __syncthreads();
    KArgs* a = &kargs();
    asm volatile("" : "+s"(a));
    const Header h = load_header(a);
    int64_t tile;
    const int unit = find_unit(a, h, w, tile);
    const uint32_t info = cld(a->unit_info, unit);
    const int k = (int)unit_info_k(info), base = (int)unit_info_base(info);
    const int c = (int)unit_info_act8(info);  // members per wave and round
    const Place at = find_place<TE>(h, 0, tile);
    const int64_t tile_byte = at.e_tile * esize;
    const int bytes = at.elems * esize;
    const bool odd = BF16 && (bytes & 2);
    const int per_round = c * (int)(blockDim.x / kBlock);
    Members m;
    for (int j0 = wave * c; j0 < k; j0 += per_round) {
      const int n = k - j0 < c ? k - j0 : c;
      wide_members<true, MOM>(a, h, base + j0, at.seg, tile_byte, m);
      // the members' flags: bits base + j0 .. of the position-ordered mask
      const int bit = base + j0;
      const uint64_t two = cld(a->member_act, bit >> 5) |
                           ((uint64_t)cld(a->member_act, (bit >> 5) + 1) << 32);
      m.act = (uint32_t)(two >> (bit & 31)) & ((1u << n) - 1u);
      u32x4 wv[kWideC], gv[kWideC], vv[kWideC];
#pragma unroll
      for (int j = 0; j < kWideC; ++j) {
        if (j < n) wv[j] = bld16(tile_rsrc(m.w[j], load_bytes(bytes)), off);
        if (m.active(j)) {
          gv[j] = bld16(tile_rsrc(m.g[j], load_bytes(bytes)), off);
          if constexpr (MOM) vv[j] = bld16(tile_rsrc(m.v[j], load_bytes(bytes)), off);
        }
      }
      asm volatile("" : "+s"(m.act));
      float x[kWideC][N];
#pragma unroll
      for (int j = 0; j < kWideC; ++j) {
        if (j < n) V::unpack(wv[j], x[j]);
        if (m.active(j)) {
          float g[N], v[N];
          V::unpack(gv[j], g);
          if constexpr (MOM) V::unpack(vv[j], v);
#pragma unroll
          for (int i = 0; i < N; ++i) x[j][i] = update<MOM, EXT>(x[j][i], g[i], v[i], h.opt);
          if constexpr (MOM) vv[j] = V::pack(v);
        }
        __builtin_amdgcn_sched_barrier(0);  // one member at a time: fewer registers
      }
      if constexpr (MOM) {
        asm volatile("" : "+s"(m.act));
#pragma unroll
        for (int j = 0; j < kWideC; ++j)
          if (m.active(j)) {
            bst16(tile_rsrc(m.v[j], bytes & ~3), off, vv[j]);
            if (odd) odd_store<1>(m.v[j], bytes, [&](int) { return vv[j]; });
          }
      }
      // The sum, from the wave that holds the members before these.
      const uint32_t turn = (uint32_t)(j0 / c);
      float s[N];
      if (turn > 0) {
        wait_turn(&sh.turn, turn);
#pragma unroll
        for (int i = 0; i < N; ++i) s[i] = sh.sum[i][lane] + x[0][i];
      } else {
#pragma unroll
        for (int i = 0; i < N; ++i) s[i] = x[0][i];
      }
#pragma unroll
      for (int j = 1; j < kWideC; ++j)
        if (j < n) {
#pragma unroll
          for (int i = 0; i < N; ++i) s[i] = s[i] + x[j][i];
        }
      if (j0 + n < k) {
#pragma unroll
        for (int i = 0; i < N; ++i) sh.sum[i][lane] = s[i];
        pass_turn(&sh.turn, turn + 1);
      } else {
        const float inv_k = kInv.v[k];
#pragma unroll
        for (int i = 0; i < N; ++i) s[i] = s[i] * inv_k;
        sh.mean[lane] = V::pack(s);
        pass_turn(&sh.turn, kWideDone);
      }
    }
    wait_turn(&sh.turn, kWideDone);
    const u32x4 out = sh.mean[lane];
    for (int j0 = wave * c; j0 < k; j0 += per_round) {
      const int n = k - j0 < c ? k - j0 : c;
      wide_members<false, MOM>(a, h, base + j0, at.seg, tile_byte, m);
#pragma unroll
      for (int j = 0; j < kWideC; ++j)
        if (j < n) {
          bst16(tile_rsrc(m.w[j], bytes & ~3), off, out);
          if (odd) odd_store<1>(m.w[j], bytes, [&](int) { return out; });
        }
    }
    if (h.blocks == 0) return;
    w += h.blocks;
    if (w >= h.work) return;
    __syncthreads();
  }
}

}  // namespace

namespace {
template <bool BF16, bool MOM>
const void* kernel_for(bool ext, bool wide) {
  if (wide)
    return ext ? reinterpret_cast<const void*>(&wide_step_kernel<BF16, MOM, true>)
               : reinterpret_cast<const void*>(&wide_step_kernel<BF16, MOM, false>);
  return ext ? reinterpret_cast<const void*>(&fused_step_kernel<BF16, MOM, true>)
             : reinterpret_cast<const void*>(&fused_step_kernel<BF16, MOM, false>);
}
}  // namespace

hipError_t launch_step(const StepArgs& a, bool bf16, bool mom, bool ext, int wide_waves,
                       size_t cu_share, hipStream_t stream) {
  const bool wide = wide_waves > 0;
  const void* fn = bf16 ? (mom ? kernel_for<true, true>(ext, wide) : kernel_for<true, false>(ext, wide))
                        : (mom ? kernel_for<false, true>(ext, wide)
                               : kernel_for<false, false>(ext, wide));
  void* args[] = {const_cast<StepArgs*>(&a)};
  const dim3 grid = a.blocks ? dim3(a.blocks) : dim3(a.work / a.n_units, a.n_units);
  // The dynamic LDS is a reservation only: it caps how many workgroups share
  // a CU.
  const size_t own = wide ? sizeof(WideShared) : 0;
  const size_t lds = cu_share > own ? cu_share - own : 0;
  // hipLaunchKernel reports this launch's own status (not an earlier sticky error).
  return hipLaunchKernel(fn, grid, dim3(wide ? kBlock * wide_waves : kBlock), args, lds, stream);
}

}  // namespace rip
