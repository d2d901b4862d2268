// liblce: linear-cross-entropy (LCE) forward and backward for MI355X (gfx950).
//
// The objective is the paper's Linear Cross-Entropy loss (Sec. 4.2): the final
// output projection H W^T is fused with the cross-entropy over the whole
// vocabulary, ignored targets are dropped before the projection, and the dense
// [tokens, vocab] logits never exist. The result equals the standard
// cross-entropy (Sec. 3.3). The ABI, its conventions and its error codes are
// documented in include/lce.h.
//
// Path (all kernels enqueue on the caller's stream, no host synchronisation):
//   forward : compact -> gather the valid rows Hv -> fwd_tile (bf16 MFMA tiles of
//             S^T = W Hv^T, each reduced to a (max, sum-exp) partial per token) ->
//             combine (merge partials, target logit, per-row loss) -> loss (fixed-order
//             reduction)
//   backward: compact -> gather Hv (both skipped when the forward's are reused) -> per
//             vocabulary slab: G tile (recompute S^T, G = c (softmax - onehot)),
//             dH32 (+)= G W_slab (K split into parts where a launch would leave CUs idle),
//             dW slab = G^T Hv (one launch with dH where few tiles would leave CUs idle) ->
//             finalise dH (parts added in order)
// Built on the same kernels: the backward with an AdamW step on each finished dW block
// (paper Sec. 4.1), a vocabulary-shard (loss-parallel) forward / combine / backward, and a
// fused linear knowledge-distillation loss whose G kernel takes the teacher's probabilities
// as soft targets.
//
// Every contraction C = A B^T (C [M, N], sum over K) runs one MFMA main loop: bf16
// v_mfma_f32_32x32x16 with fp32 accumulation, waves of 128x64 outputs, K streamed through
// two 64-wide LDS slices filled by direct-to-LDS buffer loads (XOR-swizzled 16-byte
// chunks). Tiles are 384x256 with 12 waves (three per SIMD) for the LCE contractions (the last round of
// a forward or G launch may take parts of them), and 256x256 with 8 waves for the distillation student
// and teachers with Dt % 64 != 0. Each operand is either K-contiguous (W and Hv in the forward and G
// kernels; G in dH) or K-major (G and Hv in dW, the W slab in dH: the MFMA fragments then come from
// transposing LDS reads), so G is written once, token-major, and W is never copied.
//
// Launch shapes follow the 8 XCDs, each with its own L2 (workgroups are dealt to them round-
// robin): the forward and G tiles go in vocabulary groups a multiple of 8 tiles wide, so that each
// XCD keeps its own W tiles while the token tiles pass (xcd_tile); the dH and dW tiles are cut into
// balanced per-XCD shares walked in bands of 4 row tiles; and the backward slab width is chosen so
// that the dW launches fill whole rounds of the 256 CUs (whole_round_slab). Which workgroup takes which
// tile is in tiles.h.

#include <hip/hip_runtime.h>

#include <math.h>
#include <stdint.h>
#include <string.h>

#include <algorithm>
#include <mutex>
#include <type_traits>
#include <utility>
#include <vector>

#include "lce.h"

#define LCE_HD __host__ __device__ __forceinline__
#include "tiles.h"

// Workspace of lce_forward_noalloc: device memory of the code object itself, one copy per GPU,
// held until the process ends. In host code `scratch` is only a stand-in for the symbol; its
// device address comes from hipGetSymbolAddress (see noalloc_scratch).
static __device__ __align__(256) char scratch[LCE_NOALLOC_SCRATCH_BYTES];

namespace {

using namespace lce_tiles;

typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));
typedef float f32x16_t __attribute__((ext_vector_type(16)));
typedef int i32x4_t __attribute__((ext_vector_type(4)));
typedef unsigned int u32x2_t __attribute__((ext_vector_type(2)));
typedef short s16x4_t __attribute__((ext_vector_type(4)));
typedef short s16x8_t __attribute__((ext_vector_type(8)));
typedef __attribute__((address_space(3))) s16x4_t lds_s16x4_t;

constexpr int TILE = 256;         // output tile edge (rows of A and of B per workgroup)
constexpr int KPAD = 64;          // K padding granularity of the backward's staged operands
constexpr int NTHREADS = 512;     // 8 waves, two per SIMD
constexpr float kLog2e = 1.4426950408889634f;
constexpr float kLn2 = 0.6931471805599453f;
constexpr uint32_t kRsrcWord3 = 0x00020000u;  // gfx9 raw buffer: 32-bit data format

// Raw buffer descriptor: base address, stride 0, num_records = bytes. num_records is capped below
// 2^31 so that offset 2^31 is always out of range (the zero-fill trick for ragged K slices); every
// access of a tile lies within its first 2^31 bytes (checked on the host, or the descriptor is
// rebuilt per slice). Two forms: the compiler's buffer-resource type for the load builtin, and the
// 4 descriptor words (in SGPRs) for the inline-asm load.
__device__ __forceinline__ __amdgpu_buffer_rsrc_t make_rsrc(const void* base, uint64_t bytes) {
  const uint32_t n = bytes > 0x7FFFFFFFull ? 0x7FFFFFFFu : (uint32_t)bytes;
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(base), (short)0, (int)n, (int)kRsrcWord3);
}

__device__ __forceinline__ i32x4_t make_rsrc_words(const void* base, uint64_t bytes) {
  const uint64_t a = (uint64_t)(uintptr_t)base;
  const uint32_t n = bytes > 0x7FFFFFFFull ? 0x7FFFFFFFu : (uint32_t)bytes;
  i32x4_t w;
  w.x = __builtin_amdgcn_readfirstlane((int)(uint32_t)a);
  w.y = __builtin_amdgcn_readfirstlane((int)((a >> 32) & 0xFFFFu));
  w.z = __builtin_amdgcn_readfirstlane((int)n);
  w.w = (int)kRsrcWord3;
  return w;
}

typedef __attribute__((address_space(3))) void lds_void_t;

// One direct-to-LDS load: 16 bytes per lane from the buffer at voffset + soffset into LDS at lds
// + 16 * lane (lds wave-uniform; m0 is its LDS byte address).
//  kAsm = false: the compiler builtin. The compiler tracks it as an LDS write and, before any LDS
//    read it cannot prove disjoint, waits for every such load in flight; it proves this for the
//    128-bit fragment reads but not for the transposing reads.
//  kAsm = true: inline asm, which the compiler does not track, for the main loops that use
//    transposing reads (a compiler wait there would stall each substep on the next slice's
//    loads). The main loop orders the loads against the reads itself: a vmcnt wait and a barrier
//    before a buffer is read, and a buffer is refilled only after the barrier that follows its
//    last read. The s_nop is the wait state an M0 write needs before a load that writes LDS.
template <bool kAsm>
__device__ __forceinline__ void dma16(const __amdgpu_buffer_rsrc_t& rs, const i32x4_t& rw, const char* lds, int m0,
                                      uint32_t voffset, uint32_t soffset) {
  if constexpr (!kAsm) {
    __builtin_amdgcn_raw_ptr_buffer_load_lds(rs, (lds_void_t*)lds, 16, (int)voffset, (int)soffset, 0, 0);
  } else {
    // m0 is an input operand: the compiler sets it (and knows the value it holds afterwards)
    asm volatile("s_nop 0\n\tbuffer_load_dwordx4 %0, %1, %2 offen lds"
                 :
                 : "v"(voffset), "s"(rw), "s"(soffset), "{m0}"(m0)
                 : "memory");
  }
}

// A 16-byte global store followed by 8 wait states, in one statement. On this part a store wider
// than 8 bytes reads its data registers after it issues, and rewriting them within a few
// instructions corrupts the stored data, while the compiler keeps only one wait state there; the
// padding keeps the next instructions of the wave away from the data registers.
__device__ __forceinline__ void store16_padded(void* p, i32x4_t v) {
  asm volatile("global_store_dwordx4 %0, %1, off\n\ts_nop 7" : : "v"(p), "v"(v) : "memory");
}

// The same for a 16-byte store through a buffer resource (descriptor words rw, per-lane voffset,
// uniform soffset).
__device__ __forceinline__ void buffer_store16_padded(i32x4_t v, const i32x4_t& rw, uint32_t voffset,
                                                      uint32_t soffset) {
  asm volatile("buffer_store_dwordx4 %0, %1, %2, %3 offen\n\ts_nop 7"
               :
               : "v"(v), "v"(voffset), "s"(rw), "s"(soffset)
               : "memory");
}

__device__ __forceinline__ float bf16_to_f32(uint32_t bits16) { return __uint_as_float(bits16 << 16); }

// two floats rounded to nearest-even bf16 in one packed conversion (lo in the low half)
__device__ __forceinline__ uint32_t pack_bf16x2(float lo, float hi) {
  typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
  typedef float f32x2_t __attribute__((ext_vector_type(2)));
  return __builtin_bit_cast(uint32_t, __builtin_convertvector((f32x2_t){lo, hi}, bf16x2_t));
}

__device__ __forceinline__ uint16_t to_bf16(float x) { return __builtin_bit_cast(uint16_t, (__bf16)x); }

// ---------------------------------------------------------------------------------------------
// AdamW (decoupled weight decay, bias-corrected moments): the optimizer that paper Sec. 4.1
// runs inside the backward pass. The per-call constants are formed once on the host; the
// element update is one function shared by the fused dW epilogue and the standalone step, with
// floating-point contraction off so both give the same bits.
// ---------------------------------------------------------------------------------------------
struct AdamWConst {
  float keep;           // 1 - lr * weight_decay
  float beta1, omb1;    // beta1, 1 - beta1
  float beta2, omb2;    // beta2, 1 - beta2
  float step_size;      // lr / (1 - beta1^t)
  float inv_sqrt_bc2;   // 1 / sqrt(1 - beta2^t)
  float eps;
};

// Parameter and moments of W [V, D]: W bf16 with row stride ldw; m, v (and master, if not null)
// fp32 dense with row stride d.
struct AdamWState {
  uint16_t* W;
  int64_t ldw;
  float* m;
  float* v;
  float* master;
};

__device__ __forceinline__ void adamw_update(float& p, float& m, float& v, float g, const AdamWConst& c) {
#pragma clang fp contract(off)
  p = p * c.keep;
  m = c.beta1 * m + c.omb1 * g;
  v = c.beta2 * v + c.omb2 * (g * g);
  const float denom = sqrtf(v) * c.inv_sqrt_bc2 + c.eps;
  p = p - c.step_size * (m / denom);
}

__device__ __forceinline__ int64_t load_target(const void* t, int tbytes, int64_t i) {
  return tbytes == 8 ? ((const int64_t*)t)[i] : (int64_t)((const int32_t*)t)[i];
}

__device__ __forceinline__ float wave_sum(float x) {
  for (int m = 32; m >= 1; m >>= 1) x += __shfl_xor(x, m);
  return x;
}
// ---------------------------------------------------------------------------------------------
// MFMA main loop: acc[bi][bj] = A[128 WM x K] * B[256 x K]^T for this workgroup's (128 WM) x 256
// tile, WM = 2 (256 x 256, 8 waves, two per SIMD) or WM = 3 (384 x 256, 12 waves, three per SIMD;
// the waves of a SIMD cover each other's memory stalls with their MFMAs).
//
// The waves form a WM x 4 grid; wave w = 4 wr + wc owns output rows wr*128.. (A rows) and
// columns wc*64.. (B rows). acc[bi][bj] (bi < 4, bj < 2) is the 32x32 block (bi, bj) of that
// 128x64 wave tile; lane l, register r of a block holds row 8 (r / 4) + 4 (l / 32) + r % 4,
// column l % 32. A fragment for v_mfma_f32_32x32x16_bf16 is 8 consecutive K values of one row
// (lane l: row l % 32, K chunk l / 32 of the 16-wide substep).
//
// K streams through two LDS buffers of 64-wide slices (A 32 or 48 KB and B 32 KB per buffer),
// copied global -> LDS by buffer loads that write LDS directly, one 16-byte chunk per lane and
// 1 KB per instruction. An operand is stored in one of two ways:
//
//  * row-major (K contiguous, e.g. H [N, D], W [V, D]): a slice is 256 or 384 rows x 128 bytes; each
//    load instruction moves 8 rows (one full cache line per row, which the memory pipeline turns
//    into whole-line requests). Chunk c of row r sits at position c ^ swz(r), swz(r) = (r & 7) ^
//    ((r >> 3) & 1), so that the 128-bit fragment reads of any 8 or 16 consecutive rows hit
//    distinct banks;
//  * K-major (the tile's 256 or 384 elements contiguous, e.g. G [Nv, Vc] as the A operand of
//    G^T H, or W [V, D] as the B operand of G W): a slice is 64 K-rows x 512 or 768 bytes; each
//    load instruction moves whole lines of consecutive K-rows. For a 256-wide operand chunk c of
//    K-row k sits at position c ^ kswz(k), kswz(k) = 4 (k & 3) + 16 ((k >> 3) & 1) (the 384-wide
//    swizzle is kpos below). Fragments come from pairs of transposing reads
//    (ds_read_b64_tr_b16): in a 16-lane group, lane i reads 4 consecutive elements (8 bytes) of
//    K-row i / 4 and lane j receives element j of the group's 16 columns from K-rows 0..3; the
//    second read covers K-rows 4..7. The swizzle spreads the 4 K-rows x 64 bytes that a half-wave
//    reads over all banks.
//
// Each load picks its source chunk so that it lands in the swizzled position.
//
// Schedule of slice j (four 16-wide substeps; WM = 2 reads fragments one substep ahead, WM = 3
// just before use): after the third substep's MFMAs are issued, one barrier both publishes slice
// j+1 (its loads were issued about a slice earlier) and frees slice j's buffer, into which slice
// j+2 is then loaded while the fourth substep runs. Waves 0..3 issue their loads at the barrier,
// the others one or two substeps later (kLateGroups): on this part a whole workgroup's load
// instructions at once fill the texture-address queues and stall the issuing waves (measured:
// 3-9 % per kernel; the better delay depends on the operand stream).
//
// K must be a multiple of 8; a ragged last slice is zero-filled by pointing the lanes past K
// outside the buffer resource (buffer loads return 0 there).
// ---------------------------------------------------------------------------------------------
constexpr int KSLICE = 64;
constexpr uint32_t kOobOffset = 0x80000000u;

// Tile geometry of the main loop with WM wave rows of 4 waves, each wave BI x BJ blocks of 32 x 32 (4 x 2
// except in the partial tiles of the forward and G launches): TM rows of A by TN of B. A slice buffer
// holds the A region (TM rows x 128 bytes) followed by the B region; two buffers. 32 rows of an operand
// are one wave's share of its loads; B's are taken by the last waves where A's leave some without any.
template <int WM, int BI = 4, int BJ = 2>
struct Geo {
  static constexpr int TM = 32 * BI * WM;
  static constexpr int TN = 128 * BJ;
  static constexpr int NT = 256 * WM;
  static constexpr int AREG = TM * 128;
  static constexpr int SLICE = AREG + TN * 128;
  static constexpr int LDS = 2 * SLICE;
  static constexpr int A_WAVES = TM / 32, B_WAVES = TN / 32;
  static constexpr int B_FIRST = A_WAVES == 4 * WM ? 0 : 4 * WM - B_WAVES;
};
constexpr int kDhWM = 3;   // wave rows of the dH contraction
constexpr int kDwWM = 3;   // wave rows of the dW contraction

// One operand of the main loop, kW (256 or 384) tile rows (row-major) or tile columns (K-major)
// wide. Waves w < kW / 32 load it, 4 KB of the operand's region per wave and slice; the load of
// the q-th kilobyte reads at voffset off[.] + soffset.
//  OP_DENSE:  rsrc covers the tile's rows (rows past the tile's end read as zeros); off[0] is
//             the byte offset of row w*32 + lane/8 plus this lane's even-q chunk (odd q: the
//             neighbouring lane's); row 8q adds q * qstride (scalar) and the slice's K offset
//             2 k0 (scalar).
//  OP_GATHER: rsrc covers the source buffer; off[q] is the byte offset of the gathered row plus
//             the chunk; the K offset is added as a scalar.
//  OP_KMAJOR: base points at K-row 0, first column of the tile; rows are ld elements apart and
//             the buffer holds `bytes` bytes from base on; the buffer resource is rebuilt per slice
//             at base + k0 * ld, so offsets stay small for any buffer size. kW = 256: off[0] /
//             off[1] are the offsets for q = 0 / 1, and q = 2 / 3 read 2 qstride (four K-rows)
//             further; kW = 384: off[q] per q.
struct Operand {
  __amdgpu_buffer_rsrc_t rsrc;
  i32x4_t rwords;
  const uint16_t* base;
  int64_t ld;
  uint64_t bytes;
  uint32_t off[4];
  uint32_t qstride;
};

// How an operand is stored: row-major rows of a dense buffer, row-major rows gathered through a
// row list, or K-major.
enum OpKind { OP_DENSE = 0, OP_GATHER = 1, OP_KMAJOR = 2 };

template <int BI, int BJ>
struct FragSet {
  bf16x8_t a[BI], b[BJ];
};

// chunk this lane loads for its even-numbered rows (odd rows: ^ 1), row-major operands
__device__ __forceinline__ int lane_chunk_even() { return lane_chunk(threadIdx.x & 63); }

// K-major swizzle: position in LDS of 16-byte chunk c (of kW / 8) of K-row k, and its inverse.
//  kW = 256: c ^ (4 (k & 3) + 16 ((k >> 3) & 1));
//  kW = 384: within each group of 16 chunks c ^ 4 (k & 3), and the three groups rotated by one
//            for K-rows with bit 3 set.
// Either way the 4 K-rows x 64 bytes a half-wave reads in one transposing read land on all banks.
__device__ __forceinline__ int kswz(int k) { return ((k & 3) << 2) | (((k >> 3) & 1) << 4); }

template <int kW>
__device__ __forceinline__ int kpos(int k, int c) {
  if constexpr (kW == 256) {
    return c ^ kswz(k);
  } else {
    const int g = (c >> 4) + ((k >> 3) & 1);
    return 16 * (g >= 3 ? g - 3 : g) + ((c & 15) ^ ((k & 3) << 2));
  }
}

template <int kW>
__device__ __forceinline__ int kchunk(int k, int pos) {
  if constexpr (kW == 256) {
    return pos ^ kswz(k);
  } else {
    const int g = (pos >> 4) - ((k >> 3) & 1);
    return 16 * (g < 0 ? g + 3 : g) + ((pos & 15) ^ ((k & 3) << 2));
  }
}

// LDS byte offset, within a kW-wide K-major operand region, of this lane's first transposing read
// for the 32-column block starting at column c0 of substep 0 (the second read is 8 kW bytes
// further: 4 K-rows; substep ks adds 32 kW ks: 16 K-rows).
template <int kW>
__device__ __forceinline__ uint32_t kmajor_frag_addr(int c0) {
  const int lane = threadIdx.x & 63, g = lane >> 4, i = lane & 15;
  const int k = 8 * (g >> 1) + (i >> 2);
  const int col = c0 + 16 * (g & 1) + 4 * (i & 3);
  return (uint32_t)(k * kW * 2 + (kpos<kW>(k, col >> 3) << 4) + (col & 7) * 2);
}

template <int kW>
__device__ __forceinline__ bf16x8_t read_tr_pair(const char* p) {
  s16x8_t t;
  t.lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4_t*)p);
  t.hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4_t*)(p + 8 * kW));
  return __builtin_bit_cast(bf16x8_t, t);
}

// Per-lane LDS read addresses of one operand.
//  row-major: rk = row base | chunk of substep 0; substep ks reads at rk ^ 32 ks (the chunk index
//             (2 ks + lane / 32) ^ swz is the substep-0 chunk ^ 2 ks), block b 4096 b further.
//  K-major:   tr for block 0 (+ 32 kW ks per substep); block b (32 columns further) reads at
//             tr ^ (b << 6): within a wave's 128 or 64 columns the block index only changes bits
//             2-3 of the chunk index, which both swizzles keep as an XOR.
template <int kBlocks>
struct FragAddr {
  uint32_t rk;
  uint32_t tr;
};

template <bool kKM, int kW, int kBlocks>
__device__ __forceinline__ void frag_addr(FragAddr<kBlocks>& fa, int row0) {
  const int lane = threadIdx.x & 63;
  if constexpr (!kKM) {
    const int swz = (lane & 7) ^ ((lane >> 3) & 1);
    fa.rk = (uint32_t)((row0 + (lane & 31)) * 128) | (uint32_t)(((lane >> 5) ^ swz) * 16);
  } else {
    fa.tr = kmajor_frag_addr<kW>(row0);
  }
}

template <bool kKM, int kW, int kBlocks>
__device__ __forceinline__ void read_operand(bf16x8_t (&f)[kBlocks], const char* reg, const FragAddr<kBlocks>& fa,
                                             int ks) {
  if constexpr (!kKM) {
    // the base address is made opaque at each read, so that its per-substep variants are formed
    // next to the reads (one VALU op each) instead of being held in registers through the loop
    uint32_t rk = fa.rk;
    asm volatile("" : "+v"(rk));
    const char* p = reg + (rk ^ (uint32_t)(32 * ks));
#pragma unroll
    for (int b = 0; b < kBlocks; ++b) f[b] = *reinterpret_cast<const bf16x8_t*>(p + b * 4096);
  } else {
#pragma unroll
    for (int b = 0; b < kBlocks; ++b) f[b] = read_tr_pair<kW>(reg + (fa.tr ^ (uint32_t)(b << 6)) + ks * 32 * kW);
  }
}

template <int BI, int BJ>
__device__ __forceinline__ void mma_substep(f32x16_t (&acc)[BI][BJ], const FragSet<BI, BJ>& f) {
#pragma unroll
  for (int i = 0; i < BI; ++i)
#pragma unroll
    for (int j = 0; j < BJ; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f.a[i], f.b[j], acc[i][j], 0, 0, 0);
}

// This wave's 4 load instructions of one kW-wide operand's slice k0 (dstp = the operand's region
// + 4 KB per wave, dst its LDS byte address). Lanes that must read zeros (past K on a ragged last
// slice) point outside the buffer resource.
template <bool kAsm, int kKind, int kW, bool kMasked>
__device__ __forceinline__ void load_operand(const Operand& op, const char* dstp, int dst, int k0, int K) {
  if constexpr (kKind != OP_KMAJOR) {
    // dense: the odd-q offset of lane L is the even-q offset of lane L ^ 1 (same row, the chunk
    // with the other parity), fetched by a quad swap instead of held in a register
    const uint32_t odd =
        kKind == OP_DENSE ? (uint32_t)__builtin_amdgcn_mov_dpp((int)op.off[0], 0xB1, 0xF, 0xF, false) : 0u;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const bool ok = !kMasked || chunk_exists(threadIdx.x & 63, q, k0, K);
      const uint32_t v = kKind == OP_DENSE ? ((q & 1) ? odd : op.off[0]) : op.off[q];
      const uint32_t so = (uint32_t)k0 * 2 + (kKind == OP_DENSE ? (uint32_t)q * op.qstride : 0u);
      dma16<kAsm>(op.rsrc, op.rwords, dstp + q * 1024, dst + q * 1024, ok ? v : kOobOffset, so);
    }
  } else {
    const uint16_t* base = op.base + (int64_t)k0 * op.ld;
    const uint64_t bytes = op.bytes - (uint64_t)k0 * op.ld * 2;
    const __amdgpu_buffer_rsrc_t rs = make_rsrc(base, bytes);
    const i32x4_t rw = make_rsrc_words(base, bytes);
    const int p0 = (threadIdx.x >> 6) * 256 + (threadIdx.x & 63);   // 16-byte unit of q = 0
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const bool ok = !kMasked || k0 + (p0 + 64 * q) / (kW / 8) < K;
      const uint32_t v = kW == 256 ? op.off[q & 1] : op.off[q];
      const uint32_t so = kW == 256 ? (uint32_t)(q & 2) * op.qstride : 0u;   // off[1] holds q = 1's rows
      dma16<kAsm>(rs, rw, dstp + q * 1024, dst + q * 1024, ok ? v : kOobOffset, so);
    }
  }
}

// Point the chunks of slice k0 at or past K outside the buffer resource (row-major operands). The
// offsets are changed in place, which takes no registers beside them in the loop, so this is for the
// last slice that is loaded. (An odd-q offset of a dense operand is the neighbouring lane's even one,
// which that lane masks by the same chunk index.)
template <int kKind>
__device__ __forceinline__ void mask_tail(Operand& op, int k0, int K) {
  static_assert(kKind != OP_KMAJOR, "");
#pragma unroll
  for (int q = 0; q < (kKind == OP_DENSE ? 1 : 4); ++q)
    if (!chunk_exists(threadIdx.x & 63, q, k0, K)) op.off[q] = kOobOffset;
}

// w: this wave's index in the workgroup, a wave-uniform (scalar) value
template <bool kAsm, int kAKind, int kBKind, class G, bool kMasked>
__device__ __forceinline__ void load_slice(const Operand& A, const Operand& B, const char* buf, int bufoff, int k0,
                                           int K, int w) {
  const char* dstp = buf + w * 4096;
  const int dst = bufoff + w * 4096;   // LDS byte address (asm loads)
  constexpr int breg = G::AREG - G::B_FIRST * 4096;
  if (G::A_WAVES == G::NT / 64 || w < G::A_WAVES) load_operand<kAsm, kAKind, G::TM, kMasked>(A, dstp, dst, k0, K);
  if (G::B_FIRST ? w >= G::B_FIRST : (G::B_WAVES == G::NT / 64 || w < G::B_WAVES))
    load_operand<kAsm, kBKind, G::TN, kMasked>(B, dstp + breg, dst + breg, k0, K);
}

// s_waitcnt with only the vector-memory counter constrained (expcnt / lgkmcnt left at max)
#define LCE_WAIT_VM(n) __builtin_amdgcn_s_waitcnt((((n) & 15) | (7 << 4) | (15 << 8) | (((n) >> 4) << 14)))

// acc = A B^T for this workgroup's (128 WM) x 256 tile. WM = 2: 8 waves, fragments double-
// buffered (read one substep ahead). WM = 3: 12 waves (three per SIMD), 384 A rows, fragments
// single-buffered (the 168 registers a wave may hold at three waves per SIMD leave no room for a
// second set; the other two waves of the SIMD cover the read latency).
// kTail (row-major operands): K is not a multiple of 64; the last slice's chunks past K read zeros.
template <int kLateGroups, int kAKind = OP_DENSE, int kBKind = OP_GATHER, int WM = 2, bool kRagged = true,
          bool kTail = false, int BI = 4, int BJ = 2>
__device__ __forceinline__ void mma_mainloop(f32x16_t (&acc)[BI][BJ], Operand A, Operand B, int K,
                                             char* smem) {
  using G = Geo<WM, BI, BJ>;
  constexpr bool kAKM = kAKind == OP_KMAJOR, kBKM = kBKind == OP_KMAJOR;
  const int wave = threadIdx.x >> 6;
  const int wr = wave >> 2, wc = wave & 3;
  static_assert((BI == 4 && BJ == 2) || (WM == 3 && !kAKM && !kBKM), "partial tiles: row-major operands");
  FragAddr<BI> fa;
  FragAddr<BJ> fb;
  frag_addr<kAKM, G::TM>(fa, wr * 32 * BI);
  frag_addr<kBKM, G::TN>(fb, wc * 32 * BJ);
  auto read_frags = [&](FragSet<BI, BJ>& f, const char* buf, int ks) {
    read_operand<kAKM, G::TM>(f.a, buf, fa, ks);
    read_operand<kBKM, G::TN>(f.b, buf + G::AREG, fb, ks);
  };

#pragma unroll
  for (int i = 0; i < BI; ++i)
#pragma unroll
    for (int j = 0; j < BJ; ++j) acc[i][j] = (f32x16_t){};

  const int S = (K + KSLICE - 1) / KSLICE;
  if (S <= 0) return;
  // kRagged = false: the caller guarantees K % 64 == 0
  const bool ragged = kRagged && (K % KSLICE) != 0;
  // loads as inline asm where transposing reads are used (see dma16)
  constexpr bool kAsm = kAKM || kBKM;
  const int lds0 = kAsm ? __builtin_amdgcn_readfirstlane((int)(uint32_t)(uintptr_t)smem) : 0;
  // One scalar copy of the wave index for the whole loop. Opaque to the compiler, so that it is
  // not recomputed from the work-item id register inside the loop: under register pressure that
  // register is spilled, and its reload would wait for every load in flight.
  int wsc = __builtin_amdgcn_readfirstlane(wave);
  asm volatile("" : "+s"(wsc));
  auto load = [&](int s) {
    char* buf = smem + (s & 1) * G::SLICE;
    const int bufoff = lds0 + (s & 1) * G::SLICE;
    if constexpr (kTail) {
      if (s == S - 1) {   // (the last slice is the last one loaded)
        mask_tail<kAKind>(A, s * KSLICE, K);
        mask_tail<kBKind>(B, s * KSLICE, K);
      }
    }
    if (ragged && s == S - 1) load_slice<kAsm, kAKind, kBKind, G, true>(A, B, buf, bufoff, s * KSLICE, K, wsc);
    else load_slice<kAsm, kAKind, kBKind, G, false>(A, B, buf, bufoff, s * KSLICE, K, wsc);
  };

  // a wave that takes a share of one operand only issues 4 loads per slice instead of 8
  const bool loads_a = G::A_WAVES == G::NT / 64 || wsc < G::A_WAVES;
  const bool loads_b = G::B_FIRST ? wsc >= G::B_FIRST : (G::B_WAVES == G::NT / 64 || wsc < G::B_WAVES);
  load(0);
  if (S > 1) {
    load(1);
    if (loads_a && loads_b) LCE_WAIT_VM(8);
    else if (loads_a || loads_b) LCE_WAIT_VM(4);
    else LCE_WAIT_VM(0);
  } else {
    LCE_WAIT_VM(0);
  }
  __builtin_amdgcn_s_barrier();

  // Waves 0..3 (the first wave of each SIMD) issue their share of a slice's loads at the barrier;
  // the others kLateGroups MFMA substeps later: a smaller load burst, and the other waves of each
  // SIMD go straight back to MFMA work.
  // slot of this wave's loads: 0 at the barrier, 1 after the slice's last substep, 2 after the
  // next slice's first substep. kLateGroups = 1 or 2: waves 4.. use that slot; 1xy (WM = 3):
  // waves 4..7 use slot x, waves 8..11 slot y.
  constexpr int kMid = kLateGroups >= 100 ? (kLateGroups / 10) % 10 : kLateGroups;
  constexpr int kLast = kLateGroups >= 100 ? kLateGroups % 10 : kLateGroups;
  const int slot = wsc < 4 ? 0 : (WM == 3 && wsc >= 8 ? kLast : kMid);
  const bool late = slot != 0;
  int pend = -1;
  if constexpr (WM == 2) {
    FragSet<BI, BJ> f0, f1;
    read_frags(f0, smem, 0);
    for (int j = 0; j < S; ++j) {
      const char* cur = smem + (j & 1) * G::SLICE;
      const char* nxt = smem + ((j + 1) & 1) * G::SLICE;
      read_frags(f1, cur, 1);
      mma_substep(acc, f0);
      if (slot == 2 && pend >= 0) {
        load(pend);
        pend = -1;
      }
      read_frags(f0, cur, 2);
      mma_substep(acc, f1);
      read_frags(f1, cur, 3);
      mma_substep(acc, f0);
      if (j + 1 < S) {
        // slice j+1 landed (own loads) and every wave is done with slice j's buffer
        __builtin_amdgcn_s_waitcnt(0);
        __builtin_amdgcn_s_barrier();
        if (j + 2 < S) {
          if (!late) load(j + 2);
          else pend = j + 2;
        }
        read_frags(f0, nxt, 0);
      }
      mma_substep(acc, f1);
      if (slot == 1 && pend >= 0) {
        load(pend);
        pend = -1;
      }
    }
  } else {
    FragSet<BI, BJ> f;
    for (int j = 0; j < S; ++j) {
      const char* cur = smem + (j & 1) * G::SLICE;
      read_frags(f, cur, 0);
      mma_substep(acc, f);
      if (slot == 2 && pend >= 0) {
        load(pend);
        pend = -1;
      }
      read_frags(f, cur, 1);
      mma_substep(acc, f);
      read_frags(f, cur, 2);
      mma_substep(acc, f);
      read_frags(f, cur, 3);
      if (j + 1 < S) {
        // slice j+1 landed (own loads) and every wave is done with slice j's buffer
        __builtin_amdgcn_s_waitcnt(0);
        __builtin_amdgcn_s_barrier();
        if (j + 2 < S) {
          if (!late) load(j + 2);
          else pend = j + 2;
        }
      }
      mma_substep(acc, f);
      if (slot == 1 && pend >= 0) {
        load(pend);
        pend = -1;
      }
    }
  }
  // every wave is done reading LDS before the caller reuses it
  __syncthreads();
}

// A row-major operand of rows [row0, row0 + kW) (tile = row0's start) of a dense buffer with
// rows_left rows from row0 on.
// (wave `first` loads the first 32 rows)
__device__ __forceinline__ Operand dense_operand(const uint16_t* tile, int rows_left, int64_t ld, int first = 0) {
  Operand op;
  op.rsrc = make_rsrc(tile, (uint64_t)rows_left * ld * 2);
  op.rwords = make_rsrc_words(tile, (uint64_t)rows_left * ld * 2);
  const int j = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int ce = lane_chunk_even();
  const uint32_t row = (uint32_t)((int64_t)((w - first) * 32 + (j >> 3)) * ld * 2);   // (used by the waves from first on)
  op.off[0] = row + ce * 16;
  op.qstride = (uint32_t)(16 * ld);   // 8 rows
  return op;
}

// kW rows n0.. of the compacted valid-row list idx[0..nv) of a buffer of n rows (rows past nv
// repeat the last valid one).
template <int kW = 256>
__device__ __forceinline__ Operand gather_operand(const uint16_t* src, int64_t n, int64_t ld, const int* idx, int n0,
                                                  int nv) {
  Operand op;
  op.rsrc = make_rsrc(src, (uint64_t)n * ld * 2);
  op.rwords = make_rsrc_words(src, (uint64_t)n * ld * 2);
  const int j = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int ce = lane_chunk_even();
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    int r = w * 32 + q * 8 + (j >> 3);
    r = n0 + (r < kW ? r : kW - 1);
    r = r < nv ? r : nv - 1;
    op.off[q] = (uint32_t)((int64_t)idx[r] * ld * 2 + (ce ^ (q & 1)) * 16);
  }
  return op;
}

// The kW rows of a row-major tile (tile = its first row) of which only the first rows_left exist,
// e.g. the last vocabulary tile of W: per-row offsets as for a gathered operand (kind OP_GATHER),
// with the rows at or past rows_left pointed at kOobOffset. No address past the existing rows is
// formed, and the loads of the missing rows return zeros.
template <int kW>
__device__ __forceinline__ Operand masked_dense_operand(const uint16_t* tile, int rows_left, int64_t ld) {
  Operand op;
  op.rsrc = make_rsrc(tile, (uint64_t)rows_left * ld * 2);
  op.rwords = make_rsrc_words(tile, (uint64_t)rows_left * ld * 2);
  const int j = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int ce = lane_chunk_even();
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    int r = w * 32 + q * 8 + (j >> 3);
    r = r < kW ? r : kW - 1;   // (waves that do not load this operand)
    op.off[q] = r < rows_left ? (uint32_t)((int64_t)r * ld * 2 + (ce ^ (q & 1)) * 16) : kOobOffset;
  }
  return op;
}

// A kW-wide K-major operand: K-row 0 of the tile at `base` (its first column), rows `ld` elements
// apart, `bytes` readable bytes from base on, and `cols` columns from base on that exist (the
// lanes whose chunk lies at or past them load from kOobOffset: zeros, and no address past a
// row's existing columns).
template <int kW = 256>
__device__ __forceinline__ Operand kmajor_operand(const uint16_t* base, int64_t ld, uint64_t bytes, int cols) {
  Operand op;
  op.base = base;
  op.ld = ld;
  op.bytes = bytes;
  op.qstride = (uint32_t)(4 * ld);      // two K-rows (kW = 256)
  const int j = threadIdx.x & 63, w = threadIdx.x >> 6;
#pragma unroll
  for (int q = 0; q < (kW == 256 ? 2 : 4); ++q) {
    int p = w * 256 + q * 64 + j;                       // 16-byte unit of the region
    p = p < kW * 8 ? p : kW * 8 - 1;                    // (waves that do not load this operand)
    const int k = p / (kW / 8), pos = p % (kW / 8);
    const int c = kchunk<kW>(k, pos);
    // kW = 256: the K-rows 4 further (q = 2, 3) have the same chunk (same bits 0-1 and 3 of k)
    op.off[q] = c * 8 < cols ? (uint32_t)((int64_t)k * ld * 2 + (c << 4)) : kOobOffset;
  }
  return op;
}

// ---------------------------------------------------------------------------------------------
// K1: valid-row compaction: the LCE objective drops ignored targets before the projection
// (Sec. 4.2), so no MFMA work is spent on their rows.
// idx[0..Nv) = ascending rows whose target is in [0, V); pos[n] = its index there or -1.
// One workgroup of 16 waves walks the rows in rounds of 1024 consecutive rows (coalesced target
// loads, up to 16 rounds loaded ahead): a row's index is the valid rows of earlier rounds, of
// earlier waves of its round (wave ballots summed through LDS) and of lower lanes of its wave
// (popcount of its ballot), so idx comes out sorted.
// ---------------------------------------------------------------------------------------------
__global__ __launch_bounds__(1024) void k_compact(const void* targets, int tbytes, int64_t n, int64_t v,
                                                  int ignore, int* idx, int* pos, int* nv_ws,
                                                  int* nv_user, int* status, float* lse_zero,
                                                  float* loss_zero, float* zero3) {
  constexpr int kAhead = 16;
  __shared__ int wsum[2][16];
  __shared__ int bad_any;
  const int t = threadIdx.x, lane = t & 63, w = t >> 6;
  if (t == 0) bad_any = 0;
  __syncthreads();
  int base = 0, bad = 0;
  for (int64_t g0 = 0; g0 < n; g0 += (int64_t)1024 * kAhead) {
    int64_t tg[kAhead];
#pragma unroll
    for (int r = 0; r < kAhead; ++r) {
      const int64_t i = g0 + (int64_t)r * 1024 + t;
      tg[r] = i < n ? load_target(targets, tbytes, i) : (int64_t)ignore;
    }
#pragma unroll
    for (int r = 0; r < kAhead; ++r) {
      const int64_t i = g0 + (int64_t)r * 1024 + t;
      if (g0 + (int64_t)r * 1024 >= n) break;   // uniform
      const bool ign = tg[r] == (int64_t)ignore;
      const bool ok = i < n && !ign && tg[r] >= 0 && tg[r] < v;
      bad |= (i < n && !ign && !ok);
      const unsigned long long m = __ballot(ok);
      const int below = __popcll(m & ((1ull << lane) - 1ull));
      if (lane == 0) wsum[r & 1][w] = __popcll(m);
      __syncthreads();   // (the buffer written here was last read two rounds ago, before a barrier)
      int before = base, total = 0;
#pragma unroll
      for (int k = 0; k < 16; ++k) {
        const int c = wsum[r & 1][k];
        before += k < w ? c : 0;
        total += c;
      }
      if (i < n) {
        if (ok) {
          const int o = before + below;
          idx[o] = (int)i;
          pos[i] = o;
        } else {
          pos[i] = -1;
          if (lse_zero) lse_zero[i] = 0.0f;
          if (loss_zero) loss_zero[i] = 0.0f;
          if (zero3) zero3[i] = 0.0f;
        }
      }
      base += total;
    }
  }
  if (bad) bad_any = 1;  // benign same-value race
  __syncthreads();
  if (t == 0) {
    *nv_ws = base;
    if (nv_user) *nv_user = base;
    if (status) *status = bad_any ? LCE_STATUS_TARGET_OUT_OF_RANGE : 0;
  }
}

// ---------------------------------------------------------------------------------------------
// K2: forward statistics. The objective (Sec. 4.2) needs each valid row's log-sum-exp over the
// whole vocabulary; here it is accumulated tile by tile from logits that are never stored (this
// library's design: the paper states the objective, not an algorithm for it). One 384-id x 256-token tile
// per workgroup of 12 waves, H given as the gathered valid rows Hv: a tile's S^T = W_tile H^T runs a
// token's logits down a lane's registers, and each tile writes one partial pair (max, sum of exp) per
// token in log2 units, part[row * npad + token], merged by K3. Widths that are not a multiple of 64
// (kTail) take the same tiles with both operands masked in the last slice: 2999 x
// 1000 x 32003 (2549 valid) forward 237 -> 172 us against 256 x 256 tiles of 8 waves that gathered rows
// in the loop.
// ---------------------------------------------------------------------------------------------
// Tiles are taken in the order of xcd_tile (tiles.h), in groups of gw vocabulary tiles (the slab
// rule's width, within the MALL cap, a multiple of 8) by all token tiles, ids fastest: the group's
// W rows stay in the MALL while the token tiles pass, and the workgroups resident on one XCD share
// their W and H tiles through its L2 as in the backward's G launches. One launch covers vt_launch tiles from
// tm0 on and writes one partial row per tile (row tm - tm0). When the rows of all tiles would take too
// much space (plan_forward), the host launches one group at a time instead: group g writes to one of two
// row sets (by the parity of g), and in launch g >= 1 the workgroup of the group's first tile of each token
// tile first folds the other set (group g - 1, complete since launches on a stream run in order) into a
// running pair per token. The workspace thus stays independent of V.
__device__ __forceinline__ void merge_pair(float& m, float& s, float m2, float s2) {
  const float mn = fmaxf(m, m2);
  if (mn == -INFINITY) return;
  s = (m == -INFINITY ? 0.f : s * exp2f(m - mn)) + (m2 == -INFINITY ? 0.f : s2 * exp2f(m2 - mn));
  m = mn;
}

// The same with a sum weighted by the same exponentials carried along (distillation).
__device__ __forceinline__ void merge_weighted(float& m, float& s, float& q, float m2, float s2, float q2) {
  const float mn = fmaxf(m, m2);
  const float a = m == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(m - mn);
  const float b = m2 == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(m2 - mn);
  s = s * a + s2 * b;   // (both sums are 0 where both maxima are -infinity)
  q = q * a + q2 * b;
  m = mn;
}

// The forward statistics of one tile or part: ids of the vleft rows of W from wt on, the tleft tokens of Hv
// from ht on; one partial pair per token to out_m / out_s.
template <bool kTail, int BI, int BJ>
__device__ __forceinline__ void fwd_part(char* smem, const uint16_t* wt, int64_t ldw, int vleft, const uint16_t* ht,
                                         int64_t ldh, int tleft, int d, float* __restrict__ out_m,
                                         float* __restrict__ out_s, float scale2) {
  constexpr int WM = 3;
  using G = Geo<WM, BI, BJ>;
  constexpr int TM = G::TM, TN = G::TN;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, wr = wave >> 2, wc = wave & 3;
  const Operand opb = dense_operand(ht, tleft, ldh, G::B_FIRST);
  f32x16_t acc[BI][BJ];
  // (kTail: d % 64 != 0); the last vocabulary tile may hold fewer than TM rows of W
  if (vleft >= TM)
    mma_mainloop<1, OP_DENSE, OP_DENSE, WM, false, kTail, BI, BJ>(acc, dense_operand(wt, vleft, ldw), opb, d, smem);
  else
    mma_mainloop<1, OP_GATHER, OP_DENSE, WM, false, kTail, BI, BJ>(acc, masked_dense_operand<TM>(wt, vleft, ldw), opb, d,
                                                                   smem);
  // the main loop ends with a barrier: its LDS is free for the wave rows' pairs [3][TN] (m, s)
  float* red_m = reinterpret_cast<float*>(smem);
  float* red_s = red_m + WM * TN;

  // rows (vocabulary ids) of this lane: 32 (BI wr + bi) + 8 (r/4) + 4 (lane/32) + r%4
  const int vb = wr * 32 * BI + (lane >> 5) * 4;
  // the rows past V of the last vocabulary tile drop out of the max and the sum; every other tile
  // takes a path with no per-element test (a runtime test would be kept, as masks, on every tile)
  auto mask_rows = [&](auto kRagged) {
    if constexpr (decltype(kRagged)::value) {
#pragma unroll
      for (int i = 0; i < BI; ++i)
#pragma unroll
        for (int j = 0; j < BJ; ++j)
#pragma unroll
          for (int r = 0; r < 16; ++r)
            if (vb + i * 32 + (r >> 2) * 8 + (r & 3) >= vleft) acc[i][j][r] = -INFINITY;
    }
  };
  if (vleft < TM) mask_rows(std::true_type{});
#pragma unroll
  for (int j = 0; j < BJ; ++j) {
    float mx = -INFINITY;
#pragma unroll
    for (int i = 0; i < BI; ++i)
#pragma unroll
      for (int r = 0; r < 16; ++r) mx = fmaxf(mx, acc[i][j][r]);
    const float nm = mx * scale2;
    float st = 0.f;
    if (nm != -INFINITY) {
#pragma unroll
      for (int i = 0; i < BI; ++i)
#pragma unroll
        for (int r = 0; r < 16; ++r) st += __builtin_amdgcn_exp2f(fmaf(acc[i][j][r], scale2, -nm));
    }
    // merge the two lane halves (disjoint ids of the same tokens)
    const float om = __shfl_xor(nm, 32), os = __shfl_xor(st, 32);
    const float mm = fmaxf(nm, om);
    float sm = 0.f;
    if (mm != -INFINITY) {
      sm = (nm == -INFINITY ? 0.f : st * __builtin_amdgcn_exp2f(nm - mm)) +
           (om == -INFINITY ? 0.f : os * __builtin_amdgcn_exp2f(om - mm));
    }
    if (lane < 32) {
      const int t = wr * TN + wc * 32 * BJ + j * 32 + lane;
      red_m[t] = mm;
      red_s[t] = sm;
    }
  }
  __syncthreads();
  // merge the three wave rows in order; one thread per token of the tile
  if (threadIdx.x < TN) {
    const int t = threadIdx.x;
    float m = red_m[t], s = red_s[t];
#pragma unroll
    for (int q = 1; q < WM; ++q) {
      const float m2 = red_m[q * TN + t], s2 = red_s[q * TN + t];
      const float mn = fmaxf(m, m2);
      if (mn != -INFINITY)
        s = (m == -INFINITY ? 0.f : s * __builtin_amdgcn_exp2f(m - mn)) +
            (m2 == -INFINITY ? 0.f : s2 * __builtin_amdgcn_exp2f(m2 - mn));
      m = mn;
    }
    if (t < tleft) {
      out_m[t] = m;
      out_s[t] = s;
    }
  }
}

// split: the last round's tiles may be cut; the partial rows are then two sets of vt_launch, tile tl writing
// row tl (the first half of its ids, or all) and row vt_launch + tl (the second half, or an empty pair).
template <bool kTail>
__global__ __launch_bounds__(Geo<3>::NT, 3) void k_fwd_tile(const uint16_t* __restrict__ W, int64_t ldw, int v,
                                                            const uint16_t* __restrict__ Hv, int64_t ldh,
                                                            const int* __restrict__ nv_ptr, int d, int tm0,
                                                            int vt_launch, int gw, int split,
                                                            float* __restrict__ part_m, float* __restrict__ part_s,
                                                            const float* __restrict__ prev_m,
                                                            const float* __restrict__ prev_s, int wprev,
                                                            float* __restrict__ run_m, float* __restrict__ run_s,
                                                            int run_init, int npad, float scale2) {
  constexpr int TM = Geo<3>::TM;
  __shared__ __attribute__((aligned(16))) char smem[Geo<3>::LDS];
  const int nv = *nv_ptr;
  if (nv == 0) return;
  const int nt = (nv + TILE - 1) / TILE;
  TilePart p;   // p.tm: launch-relative vocabulary tile
  if (!tile_part((int)blockIdx.x, vt_launch, gw, nt, split, p)) return;
  const int tl = p.tm, n0 = p.tn * TILE;
  const int v0 = (tm0 + tl) * TM, vleft = v - v0;
  if (prev_m && tl == 0 && threadIdx.x < TILE) {   // (launches with a previous group are not split)
    const int tok = n0 + threadIdx.x;
    if (tok < nv) {
      float m = -INFINITY, s = 0.f;
      if (!run_init) {
        m = run_m[tok];
        s = run_s[tok];
      }
#pragma unroll 8
      for (int q = 0; q < wprev; ++q) merge_pair(m, s, prev_m[(int64_t)q * npad + tok], prev_s[(int64_t)q * npad + tok]);
      run_m[tok] = m;
      run_s[tok] = s;
    }
  }
  float* om = part_m + (int64_t)tl * npad + n0;
  float* os = part_s + (int64_t)tl * npad + n0;
  // (a token tile of at most 128 valid tokens takes a tile half as wide: 1364 tokens of 3584 x 152064, whose
  // last of six token tiles holds 84, forward 1290 -> 1255 us and G 1330 -> 1240; 285 of 2048 x 128256 205 ->
  // 190 and 238 -> 213)
  if (p.parts == 1) {
    if (nv - n0 > TILE / 2)
      fwd_part<kTail, 4, 2>(smem, W + (int64_t)v0 * ldw, ldw, vleft, Hv + (int64_t)n0 * ldh, ldh, nv - n0, d, om, os,
                            scale2);
    else
      fwd_part<kTail, 4, 1>(smem, W + (int64_t)v0 * ldw, ldw, vleft, Hv + (int64_t)n0 * ldh, ldh, nv - n0, d, om, os,
                            scale2);
    if (tail_parts(tile_space(vt_launch, nt), split) > 1 && threadIdx.x < TILE && n0 + (int)threadIdx.x < nv) {
      om[(int64_t)vt_launch * npad + threadIdx.x] = -INFINITY;
      os[(int64_t)vt_launch * npad + threadIdx.x] = 0.f;
    }
    return;
  }
  // a part: half of the tile's ids (none of them may exist), all or half of its tokens
  const int ih = p.part & 1, th = p.part >> 1;
  const int vl = vleft - ih * (TM / 2) > 0 ? vleft - ih * (TM / 2) : 0;
  const uint16_t* wt = W + (int64_t)(v0 + (vl > 0 ? ih * (TM / 2) : 0)) * ldw;
  om += (int64_t)ih * vt_launch * npad;
  os += (int64_t)ih * vt_launch * npad;
  if (p.parts == 2 && nv - n0 > TILE / 2) {
    fwd_part<kTail, 2, 2>(smem, wt, ldw, vl, Hv + (int64_t)n0 * ldh, ldh, nv - n0, d, om, os, scale2);
  } else {
    const int t0 = th * (TILE / 2);
    if (n0 + t0 >= nv) return;
    fwd_part<kTail, 2, 1>(smem, wt, ldw, vl, Hv + (int64_t)(n0 + t0) * ldh, ldh, nv - n0 - t0, d, om + t0, os + t0,
                          scale2);
  }
}

// ---------------------------------------------------------------------------------------------
// K3: per valid token: merge the vocabulary partials into lse, take the target logit
// s[n, t_n] = H[n] . W[t_n] in fp32, and the per-row loss l_n = lse_n - s[n, t_n].
// A workgroup of 16 waves serves kTok consecutive tokens, 16 or 64. Its waves first take the target logits of
// kTok / 16 tokens each, wave-wide dot products; then a wave's 64 / kTok groups of lanes fold a partial row each
// (reads along the tokens), and the groups and the waves are merged in a fixed order. Bound by latency (few
// tokens) or by the partials' bytes. With 64 tokens a workgroup, a wave folds a quarter as many rows in
// parallel: 496 valid tokens of 2048 x 128256 are 8 workgroups, 59 us against 20; 12288 of 4096 x 128256 73
// against 56. Many tokens of a narrow head prefer it (wide_combine).
// ---------------------------------------------------------------------------------------------
template <int kTok>
__global__ __launch_bounds__(1024) void k_combine(const uint16_t* __restrict__ H, int64_t ldh,
                                                  const uint16_t* __restrict__ W, int64_t ldw,
                                                  const void* targets, int tbytes, int64_t id0, int64_t v_local,
                                                  const int* __restrict__ idx, const int* __restrict__ nv_ptr,
                                                  int d, int tiles, int split, const float* __restrict__ part_m,
                                                  const float* __restrict__ part_s, int npad,
                                                  const float* __restrict__ run_m, const float* __restrict__ run_s,
                                                  float* __restrict__ lse_out, float* __restrict__ terms,
                                                  float* __restrict__ per_token, float* __restrict__ tgt_part) {
  // run_m / run_s (may be null): a running pair per token folded in before the partial rows (two sets where
  // the forward cut its last tiles)
  constexpr int kGroups = 64 / kTok;   // of lanes, a partial row each
  __shared__ float red_m[16][kTok], red_s[16][kTok], dots[kTok];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, t = lane % kTok;
  const int i0 = blockIdx.x * kTok;
  const int nv = *nv_ptr;
  if (i0 >= nv) return;
  // this wave's kTok / 16 tokens side by side, so that their chains of loads (row, target, operands) overlap
  constexpr int kPer = kTok / 16;
  int row_p[kPer];
  float dot_p[kPer];
#pragma unroll
  for (int p = 0; p < kPer; ++p) row_p[p] = i0 + wave * kPer + p < nv ? idx[i0 + wave * kPer + p] : -1;
  // target id relative to this W's first row (id0 > 0 only for a vocabulary shard, which may
  // not hold the target: then its target logit is 0)
  const uint4* hr[kPer];
  const uint4* wt[kPer];
  bool in[kPer], any = false;
#pragma unroll
  for (int p = 0; p < kPer; ++p) {
    const int64_t tl = row_p[p] >= 0 ? load_target(targets, tbytes, row_p[p]) - id0 : -1;
    in[p] = tl >= 0 && tl < v_local;
    any |= in[p];
    hr[p] = reinterpret_cast<const uint4*>(H + (int64_t)(in[p] ? row_p[p] : 0) * ldh);
    wt[p] = reinterpret_cast<const uint4*>(W + (in[p] ? tl : 0) * ldw);
    dot_p[p] = 0.f;
  }
  if (any) {
    // two chunks in flight: with four, the registers leave one workgroup a CU (16384 x 1024 x 128256 39 us, so 29;
    // 700 x 4096 x 5000 10.0 against 10.4)
#pragma unroll kPer == 1 ? 2 : 1
    for (int c = lane; c < d / 8; c += 64) {
#pragma unroll
      for (int p = 0; p < kPer; ++p) {
        if (kPer > 1 && !in[p]) continue;
        const uint4 a = hr[p][c], b = wt[p][c];
        const uint32_t av[4] = {a.x, a.y, a.z, a.w}, bv[4] = {b.x, b.y, b.z, b.w};
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          dot_p[p] = fmaf(bf16_to_f32(av[q] & 0xFFFF), bf16_to_f32(bv[q] & 0xFFFF), dot_p[p]);
          dot_p[p] = fmaf(bf16_to_f32(av[q] >> 16), bf16_to_f32(bv[q] >> 16), dot_p[p]);
        }
      }
    }
  }
#pragma unroll
  for (int p = 0; p < kPer; ++p) {
    const float dot = wave_sum(dot_p[p]);
    if (lane == 0) dots[wave * kPer + p] = dot;
  }
  const int i = i0 + t;
  const int rows = tail_parts(tile_space(tiles, (nv + TILE - 1) / TILE), split) > 1 ? 2 * tiles : tiles;
  float m = -INFINITY, s = 0.f;
  if (i < nv) {
    if (run_m && wave == 0 && lane < kTok) {
      m = run_m[i];
      s = run_s[i];
    }
#pragma unroll 4
    for (int q = kGroups * wave + lane / kTok; q < rows; q += 16 * kGroups)
      merge_pair(m, s, part_m[(int64_t)q * npad + i], part_s[(int64_t)q * npad + i]);
  }
  for (int o = kTok; o <= 32; o <<= 1) merge_pair(m, s, __shfl_xor(m, o), __shfl_xor(s, o));
  if (lane < kTok) {
    red_m[wave][t] = m;
    red_s[wave][t] = s;
  }
  __syncthreads();
  if (threadIdx.x >= kTok || i >= nv) return;
  for (int w = 1; w < 16; ++w) merge_pair(m, s, red_m[w][t], red_s[w][t]);
  const int row = idx[i];
  const float lse = (m + log2f(s)) * kLn2, dot = dots[t];
  lse_out[row] = lse;
  if (tgt_part) {
    tgt_part[row] = dot;
  } else {
    terms[i] = lse - dot;
    if (per_token) per_token[row] = lse - dot;
  }
}

// Combine of vocabulary shards: lse = log sum_g exp(lse_g) (max-shifted, shards in order) and the
// target logit sum_g tgt_g (one shard holds it), per valid token; one thread per token.
__global__ __launch_bounds__(256) void k_shard_combine(int g_count, const float* __restrict__ lse_parts,
                                                       const float* __restrict__ tgt_parts, int64_t ld,
                                                       const int* __restrict__ idx, const int* __restrict__ nv_ptr,
                                                       float* __restrict__ lse_out, float* __restrict__ terms,
                                                       float* __restrict__ per_token) {
  const int i = blockIdx.x * 256 + threadIdx.x;
  if (i >= *nv_ptr) return;
  const int row = idx[i];
  float mm = -INFINITY;
  for (int g = 0; g < g_count; ++g) mm = fmaxf(mm, lse_parts[g * ld + row]);
  float se = 0.f, z = 0.f;
  for (int g = 0; g < g_count; ++g) {
    se += exp2f((lse_parts[g * ld + row] - mm) * kLog2e);
    z += tgt_parts[g * ld + row];
  }
  const float lse = mm + log2f(se) * kLn2;
  lse_out[row] = lse;
  terms[i] = lse - z;
  if (per_token) per_token[row] = lse - z;
}

// K3b: loss = sum or mean of the per-row terms, fixed-order fp64 tree.
__global__ __launch_bounds__(1024) void k_loss(const float* __restrict__ terms, const int* __restrict__ nv_ptr,
                                               int reduction, float* __restrict__ loss) {
  __shared__ double red[1024];
  const int t = threadIdx.x;
  const int nv = *nv_ptr;
  double s = 0.0;
  for (int i = t; i < nv; i += 1024) s += (double)terms[i];
  red[t] = s;
  __syncthreads();
  for (int w = 512; w > 0; w >>= 1) {
    if (t < w) red[t] += red[t + w];
    __syncthreads();
  }
  if (t == 0) {
    double r = red[0];
    if (nv == 0) r = 0.0;
    else if (reduction == LCE_REDUCE_MEAN) r /= (double)nv;
    *loss = (float)r;
  }
}

__global__ void k_fwd_empty(float* loss, int* nv_user, int* status) {
  if (threadIdx.x == 0) {
    if (loss) *loss = 0.f;
    *nv_user = 0;
    if (status) *status = 0;
  }
}

// ---------------------------------------------------------------------------------------------
// Hv[i][:] = H[idx[i]][:] for i < Nv (rows of d elements), zero rows up to round_up(Nv, 64): the
// valid rows of H made contiguous. It is the B operand of the backward G tiles (row-major) and of
// the dW contraction (K-major over tokens), so neither main loop gathers rows itself.
// ---------------------------------------------------------------------------------------------
__global__ __launch_bounds__(256) void k_gather_rows(const uint16_t* __restrict__ H, int64_t ldh,
                                                     const int* __restrict__ idx, const int* __restrict__ nv_ptr,
                                                     int d, uint16_t* __restrict__ Hv) {
  const int nv = *nv_ptr;
  const int64_t rows = (nv + 63) / 64 * 64;
  const int cpr = d / 8;   // 16-byte chunks per row
  const int64_t total = rows * cpr;
  for (int64_t e = (int64_t)blockIdx.x * 256 + threadIdx.x; e < total; e += (int64_t)gridDim.x * 256) {
    const int64_t i = e / cpr;
    const int c = (int)(e - i * cpr);
    uint4 v = make_uint4(0, 0, 0, 0);
    if (i < nv) v = *reinterpret_cast<const uint4*>(H + (int64_t)idx[i] * ldh + c * 8);
    *reinterpret_cast<uint4*>(Hv + i * d + c * 8) = v;
  }
}

// scale c = g / n_norm (mean) or g (sum), 0 when the count is 0; for NONE the caller reads
// the per-token gradient instead
__device__ __forceinline__ float grad_scale(const float* grad, const int* n_norm, int reduction) {
  if (reduction == LCE_REDUCE_NONE) return 0.f;
  const float g = *grad;
  if (reduction == LCE_REDUCE_SUM) return g;
  const int nn = *n_norm;
  return nn > 0 ? g / (float)nn : 0.f;
}

// ---------------------------------------------------------------------------------------------
// K4: softmax-gradient tile for one vocabulary slab. Tile (vocabulary tile tm, token tile tn) of
// S^T = W_slab Hv^T is recomputed and turned into G = c (exp(s - lse) - onehot), rounded to
// bf16 and written as G[token][v] (row stride vc). A tile, or a part of one, is written whole: entries of
// tokens at or beyond Nv and of ids at or beyond the slab width vs are zeros. Parts without such a token
// or id at all, and the second half of a last token tile of at most 128 tokens, are not written; neither
// contraction that reads G needs a mask for them:
//  - dH (K = ids) takes the rows below Nv only, and along K the 16-byte chunks that start below vs; parts are
//    192 ids, so the last chunk lies in a part that is written;
//  - dW (K = tokens, G read K-major) takes the tokens below round_up(Nv, 64), which lie in the same 128 as
//    token Nv - 1, and of the ids at or beyond vs it may read what is left there, but forms only rows of dW
//    past the slab from it, which are not stored.
// ---------------------------------------------------------------------------------------------
// One tile or part of the LCE gradient: the vleft ids from W row wt on (target of a token: id tbase), the tleft
// tokens of Hv / idx from ht / idx0 on, G from element (first token, first id) on (row stride vc).
template <bool kTail, int BI, int BJ>
__device__ __forceinline__ void g_part(char* smem, const uint16_t* wt, int64_t ldw, int vleft, const uint16_t* ht,
                                       int64_t ldh, int tleft, const void* targets, int tbytes, int64_t tbase,
                                       const int* __restrict__ idx0, const float* __restrict__ lse,
                                       const float* __restrict__ grad, const int* __restrict__ n_norm, int reduction,
                                       int d, uint16_t* __restrict__ G0, int vc) {
  using G = Geo<3, BI, BJ>;
  constexpr int TM = G::TM, TN = G::TN;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, wr = wave >> 2, wc = wave & 3;
  const Operand opb = dense_operand(ht, tleft, ldh, G::B_FIRST);
  f32x16_t acc[BI][BJ];
  // (kTail: d % 64 != 0); the last tile of the vocabulary may hold fewer than TM rows of W
  if (vleft >= TM)
    mma_mainloop<1, OP_DENSE, OP_DENSE, 3, false, kTail, BI, BJ>(acc, dense_operand(wt, vleft, ldw), opb, d, smem);
  else
    mma_mainloop<1, OP_GATHER, OP_DENSE, 3, false, kTail, BI, BJ>(acc, masked_dense_operand<TM>(wt, vleft, ldw), opb, d,
                                                                  smem);
  const float c_all = grad_scale(grad, n_norm, reduction);
  int tgt[BJ];
  float l2[BJ], cj[BJ];
#pragma unroll
  for (int j = 0; j < BJ; ++j) {
    const int t = wc * 32 * BJ + j * 32 + (lane & 31);
    if (t < tleft) {
      const int row = idx0[t];
      l2[j] = lse[row] * kLog2e;
      tgt[j] = (int)(load_target(targets, tbytes, row) - tbase);
      cj[j] = reduction == LCE_REDUCE_NONE ? grad[row] : c_all;
    } else {
      l2[j] = 0.f;
      tgt[j] = -1;
      cj[j] = 0.f;
    }
  }
  const int vb = wr * 32 * BI + (lane >> 5) * 4;  // tile-relative vocabulary row base of this lane
  // G straight from registers. A lane holds 4 consecutive ids of a token row per (block, group
  // of 8 ids), the other 4 sit in lane L ^ 32; one lane swap across the wave halves
  // (permlane32 swap) per pair of groups gives each lane 8 consecutive ids (lanes < 32 the even
  // group, the others the odd one), stored as 16 bytes. Rows of tokens >= Nv and ids >= the
  // slab width get zeros, so the whole tile is written (the slab width vc is a multiple of 384).
  const i32x4_t rg = make_rsrc_words(G0, (uint64_t)TN * vc * 2);
  const uint32_t voff = (uint32_t)(((wc * 32 * BJ + (lane & 31)) * vc + wr * 32 * BI + (lane >> 5) * 8) * 2);
  // A tile whose tokens are all valid and whose ids all lie in the slab needs no test per
  // element; on the other tiles the values out of range are replaced by zeros (a select, not a
  // branch per element: the exponential of a row past Nv may be anything, even NaN).
  auto store_tile = [&](auto kFull) {
#pragma unroll
    for (int j = 0; j < BJ; ++j) {
      const bool tok_ok = wc * 32 * BJ + j * 32 + (lane & 31) < tleft;
      // the lane's element (i, q, e) is the target's when dt == 32 i + 8 q + e: one compare
      // with a constant per element, and the one-hot term folded into the scaling fma
      const int dt = tgt[j] - vb;
      const float nc = -cj[j];
#pragma unroll
      for (int i = 0; i < BI; ++i)
#pragma unroll
        for (int p = 0; p < 2; ++p) {
          u32x2_t pk[2];
#pragma unroll
          for (int h = 0; h < 2; ++h) {
            const int q = 2 * p + h;
            float gq[4];
#pragma unroll
            for (int e = 0; e < 4; ++e) {
              const int k = i * 32 + q * 8 + e;
              const float ex = __builtin_amdgcn_exp2f(fmaf(acc[i][j][q * 4 + e], kLog2e, -l2[j]));
              float g = fmaf(cj[j], ex, dt == k ? nc : 0.f);
              if constexpr (!decltype(kFull)::value) g = (tok_ok && vb + k < vleft) ? g : 0.f;
              gq[e] = g;
            }
            pk[h].x = pack_bf16x2(gq[0], gq[1]);
            pk[h].y = pack_bf16x2(gq[2], gq[3]);
          }
          // lane L < 32: (its group 2p ids 0-3, lane L + 32's ids 4-7); lane L + 32: (lane L's
          // group 2p + 1 ids 0-3, its own ids 4-7)
          const auto sx = __builtin_amdgcn_permlane32_swap(pk[0].x, pk[1].x, false, false);
          const auto sy = __builtin_amdgcn_permlane32_swap(pk[0].y, pk[1].y, false, false);
          const i32x4_t v16 = {(int)sx[0], (int)sy[0], (int)sx[1], (int)sy[1]};
          const uint32_t so = (uint32_t)((j * 32 * vc + i * 32 + p * 16) * 2);
          // (the compiled code may rewrite v16's registers right after the store: padded)
          buffer_store16_padded(v16, rg, voff, so);
        }
    }
  };
  if (tleft >= TN && vleft >= TM) store_tile(std::true_type{});
  else store_tile(std::false_type{});
}

template <bool kTail>
__global__ __launch_bounds__(Geo<3>::NT, 3) void k_bwd_g(const uint16_t* __restrict__ W, int64_t ldw, int64_t v0, int vs,
                                                       const uint16_t* __restrict__ Hv, int64_t ldh,
                                                       const void* targets, int tbytes, int64_t id0,
                                                       const int* __restrict__ idx, const int* __restrict__ nv_ptr,
                                                       const float* __restrict__ lse, const float* __restrict__ grad,
                                                       const int* __restrict__ n_norm, int reduction, int d, int tm_count,
                                                       int gw, int split, uint16_t* __restrict__ G, int vc) {
  constexpr int TM = Geo<3>::TM;
  __shared__ __attribute__((aligned(16))) char smem[Geo<3>::LDS];
  const int nv = *nv_ptr;
  if (nv == 0) return;
  TilePart p;
  if (!tile_part((int)blockIdx.x, tm_count, gw, (nv + TILE - 1) / TILE, split, p)) return;
  const int ih = p.parts > 1 ? p.part & 1 : 0, th = p.part >> 1;
  const int n0 = p.tn * TILE + th * (TILE / 2), vt0 = p.tm * TM + ih * (TM / 2);   // slab-relative
  // (a part without ids of the slab or without valid tokens: no column or row of G that is read)
  if (n0 >= nv || vt0 >= vs) return;
  const uint16_t* wt = W + (v0 + vt0) * ldw;
  const uint16_t* ht = Hv + (int64_t)n0 * ldh;
  uint16_t* g0 = G + (int64_t)n0 * vc + vt0;
  const int64_t tbase = id0 + v0 + vt0;
  const bool wide = nv - n0 > TILE / 2;   // (else the tile's tokens fit one half as wide, and no other row is read)
  if (p.parts == 1 && wide)
    g_part<kTail, 4, 2>(smem, wt, ldw, vs - vt0, ht, ldh, nv - n0, targets, tbytes, tbase, idx + n0, lse, grad, n_norm,
                        reduction, d, g0, vc);
  else if (p.parts == 1)
    g_part<kTail, 4, 1>(smem, wt, ldw, vs - vt0, ht, ldh, nv - n0, targets, tbytes, tbase, idx + n0, lse, grad, n_norm,
                        reduction, d, g0, vc);
  else if (p.parts == 2 && wide)
    g_part<kTail, 2, 2>(smem, wt, ldw, vs - vt0, ht, ldh, nv - n0, targets, tbytes, tbase, idx + n0, lse, grad, n_norm,
                        reduction, d, g0, vc);
  else
    g_part<kTail, 2, 1>(smem, wt, ldw, vs - vt0, ht, ldh, nv - n0, targets, tbytes, tbase, idx + n0, lse, grad, n_norm,
                        reduction, d, g0, vc);
}

// The tiles of the distillation loss (KD, soft targets), in four modes:
//   Z_WRITE   teacher, forward: the logits of this slab, fp32, into P
//   KD_STATS  student, forward: per token, over the tile's ids, the (max, sum-exp) pairs of teacher and
//             student logits / T and the teacher-weighted sum of the student's logits / T (qpart)
//   P_WRITE   teacher, backward: P = softmax(z/T) of this slab, fp32
//   G_SOFT    student, backward: G = c (softmax(z/T) - P) / T
// scale2 = log2(e) / T (log2(e) for LCE), inv_t = 1 / T; lse is that of the scaled logits.
//
// The forward thus runs each head's contraction once: the weights exp(z_t/T - max) of the sum are taken
// against the maximum of the tile's ids and the sums of all tiles are merged under their common maximum
// (k_kd_combine), as the sum-exp itself. (Taken against the teacher's log-sum-exp, the sum needs both
// heads' logits again after the statistics: 3072 valid tokens, 4096 -> 2048 wide, 128256 ids: forward
// 9300 us, now 4760.)
enum KdMode { G_SOFT, KD_STATS, P_WRITE, Z_WRITE };
constexpr int kKdVals = 5;   // values per token and tile of KD_STATS: teacher max, sum, weighted sum; student max, sum

template <int kMode, int WM>
__global__ __launch_bounds__(Geo<WM>::NT, WM) void k_kd_tile(const uint16_t* __restrict__ W, int64_t ldw, int64_t v0, int vs,
                                                       const uint16_t* __restrict__ H, int64_t ldh, int64_t n,
                                                       const int* __restrict__ idx, const int* __restrict__ nv_ptr,
                                                       const float* __restrict__ lse, const float* __restrict__ grad,
                                                       const int* __restrict__ n_norm, int reduction, int d, int tm_count,
                                                       uint16_t* __restrict__ G, int vc, int ldt,
                                                       float scale2, float inv_t, float* __restrict__ P,
                                                       float* __restrict__ qpart, int gsub) {
  // 12 waves (WM = 3, 384 ids per tile) serve the teacher when Dt % 64 == 0; the student and other
  // teachers keep 8 waves (and the student's G the LDS-staged epilogue below)
  static_assert(WM == 2 || kMode == P_WRITE || kMode == Z_WRITE, "");
  constexpr int TM = Geo<WM>::TM;
  __shared__ __attribute__((aligned(16))) char smem[Geo<WM>::LDS];
  const int nv = *nv_ptr;
  // tiles in the XCD-aware order of xcd_tile, in groups of gsub id tiles (ldt = Npad: ldt / 256
  // token tiles)
  int tm, tn;
  if (!xcd_tile((int)blockIdx.x, tm_count, gsub, ldt / TILE, tm, tn)) return;
  const int n0 = tn * TILE;
  if (n0 >= nv) return;
  const int vt0 = tm * TM;                   // slab-relative
  const int vleft = vs - vt0;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, wr = wave >> 2, wc = wave & 3;

  const uint16_t* wt = W + (v0 + vt0) * ldw;
  f32x16_t acc[4][2];
  // the last tile of the vocabulary may hold fewer than TM rows of W
  if constexpr (WM == 3) {
    // H is the gathered valid rows Hv (row stride ldh = d): a dense operand; d % 64 == 0 (host)
    const Operand opb = dense_operand(H + (int64_t)n0 * ldh, nv - n0, ldh);
    if (vleft >= TM)
      mma_mainloop<1, OP_DENSE, OP_DENSE, WM, false>(acc, dense_operand(wt, vleft, ldw), opb, d, smem);
    else
      mma_mainloop<1, OP_GATHER, OP_DENSE, WM, false>(acc, masked_dense_operand<TM>(wt, vleft, ldw), opb, d, smem);
  } else {
    const Operand opb = gather_operand(H, n, ldh, idx, n0, nv);
    if (vleft >= TM)
      mma_mainloop<2, OP_DENSE, OP_GATHER, WM>(acc, dense_operand(wt, vleft, ldw), opb, d, smem);
    else
      mma_mainloop<2, OP_GATHER, OP_GATHER, WM>(acc, masked_dense_operand<TM>(wt, vleft, ldw), opb, d, smem);
  }

  // the gradient scale exists only for the modes that write G (the other passes get no upstream
  // gradient: grad and n_norm, and in the forward lse, may be null there)
  constexpr bool kWritesG = kMode == G_SOFT;
  constexpr bool kUsesLse = kWritesG || kMode == P_WRITE;
  const float c_all = kWritesG ? grad_scale(grad, n_norm, reduction) : 0.f;
  int tok[2];
  float l2[2], cj[2];
#pragma unroll
  for (int j = 0; j < 2; ++j) {
    tok[j] = n0 + wc * 64 + j * 32 + (lane & 31);
    if (tok[j] < nv) {
      const int row = idx[tok[j]];
      l2[j] = kUsesLse ? lse[row] * kLog2e : 0.f;
      cj[j] = kWritesG && reduction == LCE_REDUCE_NONE ? grad[row] : c_all;
    } else {
      l2[j] = 0.f;
      cj[j] = 0.f;
    }
  }
  const int vb = wr * 128 + (lane >> 5) * 4;  // tile-relative vocabulary row base of this lane
  // The teacher's values P of one slab lie in units of 128 ids x 64 tokens, the part of a tile that one
  // wave holds (in 12- and 8-wave tiles alike), each in the order of its accumulators: register group q of
  // block (i, j) is 1 KB, 16 bytes a lane. Producer and consumer move 16 bytes per lane and whole lines
  // (id-major rows of P took 4 bytes per lane and two 128-byte pieces per instruction).
  const int wr_u = __builtin_amdgcn_readfirstlane(wr), wc_u = __builtin_amdgcn_readfirstlane(wc);
  float* punit = P + ((int64_t)(vt0 / 128 + wr_u) * (ldt / 64) + (n0 / 64 + wc_u)) * (128 * 64);
  // The student's epilogues take block b + 1's loads in flight while they use block b = 4 j + i (kF: no test
  // per element; else `absent` stands for ids past the slab and tokens past Nv).
  auto load_teacher = [&](float (&x)[16], int b, auto kFull, float absent) {
    constexpr bool kF = decltype(kFull)::value;
    const int i = b & 3, j = b >> 2;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const float4 v = *reinterpret_cast<const float4*>(punit + ((i * 2 + j) * 4 + q) * 256 + lane * 4);
      x[4 * q] = v.x;
      x[4 * q + 1] = v.y;
      x[4 * q + 2] = v.z;
      x[4 * q + 3] = v.w;
    }
    if constexpr (!kF) {
#pragma unroll
      for (int r = 0; r < 16; ++r)
        x[r] = (tok[j] < nv && vb + i * 32 + (r >> 2) * 8 + (r & 3) < vleft) ? x[r] : absent;
    }
  };
  if constexpr (kMode == P_WRITE || kMode == Z_WRITE) {
    // the whole tile is written (the consumer masks the ids and tokens that do not exist)
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          float x[4];
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            float z = acc[i][j][4 * q + e];
            // a copy made here, store by store: the compiler forms all stores' operands at once and spills
            if constexpr (kMode == Z_WRITE) asm volatile("" : "+v"(z));
            x[e] = kMode == Z_WRITE ? z : __builtin_amdgcn_exp2f(fmaf(z, scale2, -l2[j]));
          }
          store16_padded(punit + ((i * 2 + j) * 4 + q) * 256 + lane * 4,
                         __builtin_bit_cast(i32x4_t, make_float4(x[0], x[1], x[2], x[3])));
        }
    return;
  } else if constexpr (kMode == KD_STATS) {
    // the main loop ends with a barrier: its LDS is free for the two wave rows' values [2][kKdVals][256]
    float* red = reinterpret_cast<float*>(smem);
    // (tiles of valid tokens and existing ids only test nothing per element)
    auto stats = [&](auto kFull) {
      constexpr bool kF = decltype(kFull)::value;
      float zt[2][16];
      load_teacher(zt[0], 0, kFull, -INFINITY);
#pragma unroll
      for (int j = 0; j < 2; ++j) {
        float mt = -INFINITY, st = 0.f, q = 0.f, ms = -INFINITY, ss = 0.f;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const int b = 4 * j + i;
          if (b < 7) load_teacher(zt[(b + 1) & 1], b + 1, kFull, -INFINITY);
          float mb = -INFINITY, sb = 0.f, qb = 0.f;
#pragma unroll
          for (int r = 0; r < 16; ++r) {
            if (!kF && vb + i * 32 + (r >> 2) * 8 + (r & 3) >= vleft) acc[i][j][r] = -INFINITY;
            ms = fmaxf(ms, acc[i][j][r]);
            mb = fmaxf(mb, zt[b & 1][r]);
          }
          mb *= scale2;
          // no value in the block: every exponential is 0 under any finite reference (no branch here, so
          // that the next block's loads stay in flight)
          const float ref = mb == -INFINITY ? 0.f : mb;
#pragma unroll
          for (int r = 0; r < 16; ++r) {
            const float e = __builtin_amdgcn_exp2f(fmaf(zt[b & 1][r], scale2, -ref));
            sb += e;
            if (kF || vb + i * 32 + (r >> 2) * 8 + (r & 3) < vleft) qb = fmaf(e, acc[i][j][r] * inv_t, qb);
          }
          merge_weighted(mt, st, q, mb, sb, qb);
        }
        ms *= scale2;
        const float ref = ms == -INFINITY ? 0.f : ms;
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
          for (int r = 0; r < 16; ++r) ss += __builtin_amdgcn_exp2f(fmaf(acc[i][j][r], scale2, -ref));
        // merge the two lane halves (disjoint ids of the same tokens)
        merge_weighted(mt, st, q, __shfl_xor(mt, 32), __shfl_xor(st, 32), __shfl_xor(q, 32));
        merge_pair(ms, ss, __shfl_xor(ms, 32), __shfl_xor(ss, 32));
        if (lane < 32) {
          float* o = red + wr * kKdVals * TILE + wc * 64 + j * 32 + lane;
          o[0] = mt;
          o[TILE] = st;
          o[2 * TILE] = q;
          o[3 * TILE] = ms;
          o[4 * TILE] = ss;
        }
      }
    };
    if (n0 + TILE <= nv && vleft >= TM) stats(std::true_type{});
    else stats(std::false_type{});
    __syncthreads();
    // merge the two wave rows; one thread per token of the tile
    const int t = threadIdx.x;
    if (t < TILE && n0 + t < nv) {
      const float* b = red + kKdVals * TILE;
      float mt = red[t], st = red[TILE + t], q = red[2 * TILE + t], ms = red[3 * TILE + t], ss = red[4 * TILE + t];
      merge_weighted(mt, st, q, b[t], b[TILE + t], b[2 * TILE + t]);
      merge_pair(ms, ss, b[3 * TILE + t], b[4 * TILE + t]);
      float* o = qpart + (int64_t)tm * kKdVals * ldt + n0 + t;
      o[0] = mt;
      o[ldt] = st;
      o[2 * (int64_t)ldt] = q;
      o[3 * (int64_t)ldt] = ms;
      o[4 * (int64_t)ldt] = ss;
    }
    return;
  }
  // G values in place, then the bf16 tile goes through LDS (free after the main loop) as
  // T[token][v], 512-byte rows whose 16-byte chunk c sits at c ^ (token & 31), so that the
  // token-major rows of G leave with wide coalesced stores. Within a chunk the two 8-byte halves
  // (ids 0-3, 4-7) trade places in token rows with bit 4 set: the 32 lanes of a half-wave, which
  // hold the same half of 32 consecutive token rows, then write 32 distinct 8-byte bank slots.
  char* T = smem;
  // a tile whose tokens are all valid and whose ids all lie in the slab tests nothing per element
  // (a runtime test would be kept, as masks and branches, on every tile)
  auto fill = [&](auto kFull) {
    constexpr bool kF = decltype(kFull)::value;
    float pt[2][16];
    load_teacher(pt[0], 0, kFull, 0.f);
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      const bool tok_ok = kF || tok[j] < nv;
      const int nl = wc * 64 + j * 32 + (lane & 31);
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int blk = 4 * j + i;
        if (blk < 7) load_teacher(pt[(blk + 1) & 1], blk + 1, kFull, 0.f);
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          float gq[4];
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            const int r = q * 4 + e;
            const int vr = vb + i * 32 + q * 8 + e;
            float g = 0.f;
            if (kF || (tok_ok && vr < vleft)) {
              const float e2 = __builtin_amdgcn_exp2f(fmaf(acc[i][j][r], scale2, -l2[j]));
              g = cj[j] * inv_t * (e2 - pt[blk & 1][r]);
            }
            gq[e] = g;
          }
          const int vl = vb + i * 32 + q * 8;
          u32x2_t pk;
          pk.x = pack_bf16x2(gq[0], gq[1]);
          pk.y = pack_bf16x2(gq[2], gq[3]);
          const uint32_t a = (uint32_t)(nl * 512 + ((((vl >> 3) ^ (nl & 31))) << 4) +
                                        ((((vl >> 2) & 1) ^ ((nl >> 4) & 1)) << 3));
          *reinterpret_cast<u32x2_t*>(T + a) = pk;
        }
      }
    }
  };
  if (n0 + TILE <= nv && vleft >= TM) fill(std::true_type{});
  else fill(std::false_type{});
  __syncthreads();
  // G rows, the whole tile (rows of tokens >= Nv are zeros): 16-byte chunks, one 512-byte row
  // per 32 threads
#pragma unroll 4
  for (int it = 0; it < 16; ++it) {
    const int q = threadIdx.x + NTHREADS * it;
    const int nl = q >> 5, ch = q & 31;
    i32x4_t val = *reinterpret_cast<const i32x4_t*>(T + nl * 512 + ((ch ^ (nl & 31)) << 4));
    if (nl & 16) val = (i32x4_t){val.z, val.w, val.x, val.y};
    store16_padded(G + (int64_t)(n0 + nl) * vc + vt0 + ch * 8, val);
  }
}

// K5: dW[v0 + m][dd] = sum_k G[k][m] Hv[k][dd] over k < round_up(Nv, 64), G [Npad][vc] and the
// gathered valid rows Hv [Npad][D] both read K-major (transposing LDS reads); tiles of (128 WM)
// ids x 256 hidden columns. The epilogue either writes the block in bf16 (each element once), adds it to the
// bf16 values already there, or hands each bf16-rounded element straight to the AdamW update of W (the
// in-backward step). Its accesses go through buffer resources over the tile's rows below the slab
// width (rows past it read 0 and drop their stores): a per-lane 32-bit offset and a wave-uniform
// row offset per element, so that the accumulators are nearly the only registers it holds.
enum DwMode { DW_STORE = 0, DW_ACCUMULATE = 1, DW_ADAMW = 2 };

// One dW tile (block blk of the dW grid, smem the workgroup's LDS).
template <int kMode, int WM>
__device__ __forceinline__ void dw_tile(char* smem, int blk, const uint16_t* __restrict__ G, int vc, int ldt, int vs,
                                        const uint16_t* __restrict__ Hv, int d, const int* __restrict__ nv_ptr,
                                        int tm_count, uint16_t* __restrict__ dW, int64_t v0, const AdamWState& st,
                                        const AdamWConst& oc) {
  constexpr int TM = Geo<WM>::TM;
  int tm, tn;
  if (!dw_unit(blk, tm_count, d, tm, tn)) return;
  const int m0 = tm * TM, d0 = tn * TILE;
  const int nv = *nv_ptr;
  const int kpad = ((nv + KPAD - 1) / KPAD) * KPAD;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, wr = wave >> 2, wc = wave & 3;
  // ldt = Npad: G has Npad rows of vc ids, Hv Npad rows of d hidden columns
  const Operand opa = kmajor_operand<TM>(G + m0, vc, ((uint64_t)ldt * vc - m0) * 2, vc - m0);
  const Operand opb = kmajor_operand<TILE>(Hv + d0, d, ((uint64_t)ldt * d - d0) * 2, d - d0);
  f32x16_t acc[4][2];
  mma_mainloop<1, OP_KMAJOR, OP_KMAJOR, WM, false>(acc, opa, opb, kpad, smem);

  const int rows = vs - m0 < TM ? vs - m0 : TM;             // valid id rows of this tile
  const int64_t r0 = v0 + m0;                               // its first row of W / dW
  const int dc = d0 + wc * 64 + (lane & 31);
  const int lrow = wr * 128 + (lane >> 5) * 4;              // this lane's first tile row
  const bool col_ok[2] = {dc < d, dc + 32 < d};
  // row offset (in elements of a row of `stride`) of block i, register r
  auto erow = [](int i, int r) { return i * 32 + (r >> 2) * 8 + (r & 3); };
  // on the last tile of the vocabulary, the rows past it are not accessed at all (dW and the
  // optimizer state end there)
  const bool partial = rows < TM;
  auto row_ok = [&](int i, int r) { return !partial || lrow + erow(i, r) < rows; };
  if constexpr (kMode != DW_ADAMW) {
    const __amdgpu_buffer_rsrc_t rw = make_rsrc(dW + r0 * d, (uint64_t)rows * d * 2);
    const uint32_t voff = (uint32_t)((lrow * d + dc) * 2);
    // tiles with all their rows in the vocabulary and all columns inside D test nothing per element
    auto store_tile = [&](auto kFull) {
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j) {
          if (!decltype(kFull)::value && !col_ok[j]) continue;
          float old[16];
          if constexpr (kMode == DW_ACCUMULATE) {
#pragma unroll
            for (int r = 0; r < 16; ++r) {
              const uint32_t so = (uint32_t)((erow(i, r) * d + j * 32) * 2);
              old[r] = (decltype(kFull)::value || row_ok(i, r))
                           ? bf16_to_f32(__builtin_amdgcn_raw_buffer_load_b16(rw, (int)voff, (int)so, 0))
                           : 0.f;
            }
          }
#pragma unroll
          for (int r = 0; r < 16; ++r) {
            const uint32_t so = (uint32_t)((erow(i, r) * d + j * 32) * 2);
            const float x = kMode == DW_ACCUMULATE ? old[r] + acc[i][j][r] : acc[i][j][r];
            if (decltype(kFull)::value || row_ok(i, r))
              __builtin_amdgcn_raw_buffer_store_b16(to_bf16(x), rw, (int)voff, (int)so, 0);
          }
        }
    };
    if (!partial && d0 + TILE <= d) store_tile(std::true_type{});
    else store_tile(std::false_type{});
  } else {
    // moments (and master) fp32 with row stride d, W bf16 with row stride ldw
    const __amdgpu_buffer_rsrc_t rm = make_rsrc(st.m + r0 * d, (uint64_t)rows * d * 4);
    const __amdgpu_buffer_rsrc_t rv = make_rsrc(st.v + r0 * d, (uint64_t)rows * d * 4);
    const __amdgpu_buffer_rsrc_t rp = make_rsrc(st.master ? st.master + r0 * d : st.m, st.master ? (uint64_t)rows * d * 4 : 0);
    const __amdgpu_buffer_rsrc_t rW = make_rsrc(st.W + r0 * st.ldw, (uint64_t)rows * st.ldw * 2);
    const bool has_master = st.master != nullptr;
    const uint32_t vo4 = (uint32_t)((lrow * d + dc) * 4);
    const uint32_t voW = (uint32_t)((lrow * st.ldw + dc) * 2);
    // as for the stores above: full tiles test nothing per element
    auto update_tile = [&](auto kFull) {
      constexpr bool kF = decltype(kFull)::value;
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j) {
          if (!kF && !col_ok[j]) continue;
          // four consecutive rows at a time: all their loads first, then the updates and stores
#pragma unroll
          for (int rq = 0; rq < 4; ++rq) {
            float p[4], mo[4], vo[4];
#pragma unroll
            for (int e = 0; e < 4; ++e) {
              const int row = erow(i, rq * 4 + e);
              const uint32_t s4 = (uint32_t)((row * d + j * 32) * 4);
              const uint32_t sW = (uint32_t)((row * st.ldw + j * 32) * 2);
              mo[e] = vo[e] = p[e] = 0.f;
              if (kF || row_ok(i, rq * 4 + e)) {
                mo[e] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(rm, (int)vo4, (int)s4, 0));
                vo[e] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(rv, (int)vo4, (int)s4, 0));
                p[e] = has_master ? __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(rp, (int)vo4, (int)s4, 0))
                                  : bf16_to_f32(__builtin_amdgcn_raw_buffer_load_b16(rW, (int)voW, (int)sW, 0));
              }
            }
#pragma unroll
            for (int e = 0; e < 4; ++e) {
              const int row = erow(i, rq * 4 + e);
              const uint32_t s4 = (uint32_t)((row * d + j * 32) * 4);
              const uint32_t sW = (uint32_t)((row * st.ldw + j * 32) * 2);
              if (!kF && !row_ok(i, rq * 4 + e)) continue;
              const float g = bf16_to_f32(to_bf16(acc[i][j][rq * 4 + e]));
              adamw_update(p[e], mo[e], vo[e], g, oc);
              __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(uint32_t, mo[e]), rm, (int)vo4, (int)s4, 0);
              __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(uint32_t, vo[e]), rv, (int)vo4, (int)s4, 0);
              if (has_master)
                __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(uint32_t, p[e]), rp, (int)vo4, (int)s4, 0);
              __builtin_amdgcn_raw_buffer_store_b16(to_bf16(p[e]), rW, (int)voW, (int)sW, 0);
            }
          }
        }
    };
    if (!partial && d0 + TILE <= d) update_tile(std::true_type{});
    else update_tile(std::false_type{});
  }
}

template <int kMode, int WM>
__global__ __launch_bounds__(Geo<WM>::NT, WM) void k_bwd_dw(const uint16_t* __restrict__ G, int vc, int ldt, int vs,
                                                           const uint16_t* __restrict__ Hv, int d,
                                                           const int* __restrict__ nv_ptr, int tm_count,
                                                           uint16_t* __restrict__ dW, int64_t v0,
                                                           AdamWState st, AdamWConst oc) {
  __shared__ __attribute__((aligned(16))) char smem[Geo<WM>::LDS];
  dw_tile<kMode, WM>(smem, (int)blockIdx.x, G, vc, ldt, vs, Hv, d, nv_ptr, tm_count, dW, v0, st, oc);
}

// K6: dH32[m][dd] (+)= sum_k G[m][k] Ws[k][dd] over the slab's k < vs; rows m < Nv. Ws = W + v0 ldw
// is the slab's first row, read K-major (transposing LDS reads); ws_rows = V - v0 rows follow.
// kz > 1 splits K in up to kz parts (dh_split_parts) for launches with fewer output tiles than CUs:
// part z accumulates into accumulator z, at dH32 + z (dH32b - dH32) (the parts follow each other),
// and the finalise adds the accumulators in a fixed order.
// One dH tile (block blk of the dH grid, smem the workgroup's LDS).
template <int WM>
__device__ __forceinline__ void dh_tile(char* smem, int blk, const uint16_t* __restrict__ G, int vc, int vs,
                                        const uint16_t* __restrict__ Ws, int64_t ldw, int64_t ws_rows, int d,
                                        const int* __restrict__ nv_ptr, float* __restrict__ dH32, int accumulate,
                                        int kz, float* __restrict__ dH32b, int acc_rows) {
  static_assert(Geo<WM>::TM == 384, "the tail slots and the finalise assume 384-row tiles");
  constexpr int TM = Geo<WM>::TM;
  const int nv = *nv_ptr;
  DhUnit u;
  if (!dh_unit(blk, nv, d, kz, acc_rows, u)) return;
  const int tm = u.tm, tn = u.tn;
  // the fp32 block that this unit accumulates into: tile origin, row stride, column of the tile's first column
  float* acc_tile;
  int ldacc, cb;
  if (u.slot < 0) {
    acc_tile = (u.z ? dH32 + (int64_t)u.z * (dH32b - dH32) : dH32) + (int64_t)tm * TM * d;
    ldacc = d;
    cb = tn * TILE;
  } else {
    acc_tile = dH32 + (int64_t)((nv + TM - 1) / TM) * TM * d + (int64_t)u.slot * kDhSlot;
    ldacc = TILE;
    cb = 0;
  }
  const int m0 = tm * TM, d0 = tn * TILE;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, wr = wave >> 2, wc = wave & 3;
  // K = the slab's vs ids; the last slice of a slab whose width is not a multiple of 64 is masked
  // (lanes past K load zeros), so no W row past the vocabulary is addressed.
  int k0;
  const int kzn = dh_k_range(vs, u.kz, u.z, k0);
  f32x16_t acc[4][2];
  if (kzn > 0) {
    const Operand opa = dense_operand(G + (int64_t)m0 * vc + k0, nv - m0, vc);
    const Operand opb = kmajor_operand<TILE>(Ws + (int64_t)k0 * ldw + d0, ldw, ((uint64_t)(ws_rows - k0) * ldw - d0) * 2,
                                             d - d0);
    if (kzn % KSLICE == 0)
      mma_mainloop<121, OP_DENSE, OP_KMAJOR, WM, false>(acc, opa, opb, kzn, smem);
    else
      mma_mainloop<121, OP_DENSE, OP_KMAJOR, WM, true>(acc, opa, opb, kzn, smem);
  } else {
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
      for (int j = 0; j < 2; ++j) acc[i][j] = (f32x16_t){};
  }
  // Read-modify-write of the fp32 accumulator block through a buffer resource over this tile's
  // valid rows (rows past Nv read 0 and drop their stores): one 32-bit per-lane offset and a
  // wave-uniform row offset per element, so that only the accumulators occupy registers; one
  // 32-row block (32 values per lane) at a time, its loads in flight together.
  const int rows = nv - m0 < TM ? nv - m0 : TM;
  const __amdgpu_buffer_rsrc_t rd = make_rsrc(acc_tile, (uint64_t)rows * ldacc * 4);
  const int dc = d0 + wc * 64 + (lane & 31);      // column of dH (validity)
  const uint32_t voff = (uint32_t)(((wr * 128 + (lane >> 5) * 4) * ldacc + cb + wc * 64 + (lane & 31)) * 4);
  const bool col_ok[2] = {dc < d, dc + 32 < d};
  // (a column past D would be the next row's: never touched; tiles of whole 256-column blocks
  // test nothing per element, and the first slab's tiles read nothing)
  auto rmw = [&](auto kFull, auto kAcc) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      float old[2][16];
#pragma unroll
      for (int j = 0; j < 2; ++j)
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          const uint32_t so = (uint32_t)(((i * 32 + (r >> 2) * 8 + (r & 3)) * ldacc + j * 32) * 4);
          old[j][r] = (decltype(kAcc)::value && (decltype(kFull)::value || col_ok[j]))
                          ? __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(rd, (int)voff, (int)so, 0))
                          : 0.f;
        }
#pragma unroll
      for (int j = 0; j < 2; ++j) {
        if (!decltype(kFull)::value && !col_ok[j]) continue;
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          const uint32_t so = (uint32_t)(((i * 32 + (r >> 2) * 8 + (r & 3)) * ldacc + j * 32) * 4);
          __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(uint32_t, old[j][r] + acc[i][j][r]), rd,
                                                (int)voff, (int)so, 0);
        }
      }
    }
  };
  const bool full = d0 + TILE <= d;
  if (accumulate) {
    if (full) rmw(std::true_type{}, std::true_type{});
    else rmw(std::false_type{}, std::true_type{});
  } else {
    if (full) rmw(std::true_type{}, std::false_type{});
    else rmw(std::false_type{}, std::false_type{});
  }
}

template <int WM>
__global__ __launch_bounds__(Geo<WM>::NT, WM) void k_bwd_dh(const uint16_t* __restrict__ G, int vc, int vs,
                                                        const uint16_t* __restrict__ Ws, int64_t ldw,
                                                        int64_t ws_rows, int d,
                                                        const int* __restrict__ nv_ptr,
                                                        float* __restrict__ dH32, int accumulate, int kz,
                                                        float* __restrict__ dH32b, int acc_rows) {
  __shared__ __attribute__((aligned(16))) char smem[Geo<WM>::LDS];
  dh_tile<WM>(smem, (int)blockIdx.x, G, vc, vs, Ws, ldw, ws_rows, d, nv_ptr, dH32, accumulate, kz,
              dH32b, acc_rows);
}

// K5 and K6 of one slab in one launch: dh_blocks blocks are the dH launch, the others the dW launch (neither
// reads what the other writes). Blocks start in order, so the units with the longer K start first and the
// shorter ones fill the CUs they leave idle: the launches' two partial rounds become one. With few tokens
// that is dH, whose tiles are few and run over the slab's ids, or a part of them; narrow heads with many
// tokens have few dW tiles, which run over all valid tokens and, started last, end alone (dH + dW, dH first,
// then by this rule: 16384 x 256 x 8192 394 -> 358 us; 16384 x 512 x 128256 3690 -> 2920; 32768 x 512 x 8192
// 861 -> 733; 32768 x 768 x 32768 2647 -> 2446; 8192 x 512 x 32768 560 -> 438).
template <int kMode, int WM>
__global__ __launch_bounds__(Geo<WM>::NT, WM) void k_bwd_dhdw(const uint16_t* __restrict__ G, int vc, int npad, int vs,
                                                             const uint16_t* __restrict__ Ws, int64_t ldw,
                                                             int64_t ws_rows, int d, const int* __restrict__ nv_ptr,
                                                             float* __restrict__ dH32, int accumulate, int kz,
                                                             float* __restrict__ dH32b, int acc_rows, int dh_blocks,
                                                             const uint16_t* __restrict__ Hv, int tm_count,
                                                             uint16_t* __restrict__ dW, int64_t v0) {
  static_assert(kMode != DW_ADAMW, "the optimizer step of dW updates the W rows that dH reads");
  __shared__ __attribute__((aligned(16))) char smem[Geo<WM>::LDS];
  const int b = dhdw_block((int)blockIdx.x, dh_blocks, (int)gridDim.x - dh_blocks, dw_first(*nv_ptr, kz, vs));
  if (b < dh_blocks)
    dh_tile<WM>(smem, b, G, vc, vs, Ws, ldw, ws_rows, d, nv_ptr, dH32, accumulate, kz, dH32b, acc_rows);
  else
    dw_tile<kMode, WM>(smem, b - dh_blocks, G, vc, npad, vs, Hv, d, nv_ptr, tm_count, dW, v0, AdamWState{}, AdamWConst{});
}

// K7: dH[row] = bf16(dH32[pos[row]]) for valid rows, +0.0 for the others. 8 elements per thread.
__global__ __launch_bounds__(256) void k_dh_finalize(const float* __restrict__ dH32, int64_t part, int kz,
                                                     const int* __restrict__ pos, int64_t n, int d,
                                                     uint16_t* __restrict__ dH, float* __restrict__ dHf,
                                                     int has_slabs, const int* __restrict__ nv_ptr, int acc_rows) {
  // kz > 1: the accumulators of the K parts the dH launches took, `part` elements apart, added in order;
  // with kz = 1, the slots of the tail tiles' K parts z = 1, 2, ... after part 0 (dh_tile)
  const int64_t e = ((int64_t)blockIdx.x * 256 + threadIdx.x) * 8;
  if (e >= n * d) return;
  const int64_t row = e / d;
  const int col = (int)(e - row * d);
  const int p = pos[row];
  float4 a = make_float4(0.f, 0.f, 0.f, 0.f), b = a;
  auto add = [&](const float* q) {
    const float4 a2 = *reinterpret_cast<const float4*>(q);
    const float4 b2 = *reinterpret_cast<const float4*>(q + 4);
    a = make_float4(a.x + a2.x, a.y + a2.y, a.z + a2.z, a.w + a2.w);
    b = make_float4(b.x + b2.x, b.y + b2.y, b.z + b2.z, b.w + b2.w);
  };
  if (p >= 0 && has_slabs) {
    a = *reinterpret_cast<const float4*>(dH32 + (int64_t)p * d + col);
    b = *reinterpret_cast<const float4*>(dH32 + (int64_t)p * d + col + 4);
    const int nv = *nv_ptr;
    const int tm_live = (nv + 383) / 384, dt = (d + TILE - 1) / TILE, t = tm_live * dt;
    if (kz > 1) {
      const int kzl = dh_split_parts(t, kz);
      for (int z = 1; z < kzl; ++z) add(dH32 + z * part + (int64_t)p * d + col);
    } else {
      if (dh_tail_fits(t, tm_live, d, acc_rows)) {
        const int tm = p / 384, tn = col / TILE;
        const int l = dh_band_index(tm, tn, tm_live, dt);
        int x = 0;
        while (x < 7 && dh_c0(x + 1, t) <= l) ++x;
        const int c0 = dh_c0(x, t), nmain = (dh_c0(x + 1, t) - c0) & ~31, nt = dh_c0(x + 1, t) - c0 - nmain;
        if (l - c0 >= nmain) {
          const int kzt = dh_tail_parts(nt), s0 = dh_slot0(x, t) + (l - c0 - nmain);
          const float* q = dH32 + (int64_t)tm_live * 384 * d + (int64_t)(p - tm * 384) * TILE + (col - tn * TILE);
          for (int z = 1; z < kzt; ++z) add(q + (int64_t)(s0 + (z - 1) * nt) * kDhSlot);
        }
      }
    }
  }
  if (dHf) {   // fp32 rows (a vocabulary shard's term of dH, to be summed over shards)
    store16_padded(dHf + e, __builtin_bit_cast(i32x4_t, a));
    store16_padded(dHf + e + 4, __builtin_bit_cast(i32x4_t, b));
  } else {
    store16_padded(dH + e, __builtin_bit_cast(i32x4_t,
        make_uint4(pack_bf16x2(a.x, a.y), pack_bf16x2(a.z, a.w), pack_bf16x2(b.x, b.y), pack_bf16x2(b.z, b.w))));
  }
}

__global__ __launch_bounds__(256) void k_zero16(uint4* __restrict__ p, int64_t n16) {
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (i < n16) p[i] = make_uint4(0, 0, 0, 0);
}

// Standalone AdamW step over W [V, D] with the bf16 gradient dW (dense [V, D]; null = zero
// gradient): eight consecutive elements of one row per thread and iteration, 16-byte accesses.
__global__ __launch_bounds__(256) void k_adamw(int64_t v, int d, const uint16_t* __restrict__ dW,
                                               AdamWState st, AdamWConst oc) {
  const int cpr = d >> 3;
  const int64_t total = v * cpr;
  for (int64_t q = (int64_t)blockIdx.x * 256 + threadIdx.x; q < total; q += (int64_t)gridDim.x * 256) {
    const int64_t row = q / cpr;
    const int col = (int)(q - row * cpr) * 8;
    const int64_t o = row * d + col;
    i32x4_t wv = {0, 0, 0, 0};
    if (!st.master) wv = *reinterpret_cast<const i32x4_t*>(st.W + row * st.ldw + col);
    i32x4_t gv = {0, 0, 0, 0};
    if (dW) gv = *reinterpret_cast<const i32x4_t*>(dW + o);
    float p[8], mo[8], vo[8];
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const float4 a = *reinterpret_cast<const float4*>(st.m + o + 4 * h);
      const float4 b = *reinterpret_cast<const float4*>(st.v + o + 4 * h);
      mo[4 * h] = a.x; mo[4 * h + 1] = a.y; mo[4 * h + 2] = a.z; mo[4 * h + 3] = a.w;
      vo[4 * h] = b.x; vo[4 * h + 1] = b.y; vo[4 * h + 2] = b.z; vo[4 * h + 3] = b.w;
      if (st.master) {
        const float4 c = *reinterpret_cast<const float4*>(st.master + o + 4 * h);
        p[4 * h] = c.x; p[4 * h + 1] = c.y; p[4 * h + 2] = c.z; p[4 * h + 3] = c.w;
      }
    }
    uint32_t wout[4];
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      const uint32_t w2 = (uint32_t)wv[e >> 1], g2 = (uint32_t)gv[e >> 1];
      if (!st.master) p[e] = bf16_to_f32((e & 1) ? (w2 >> 16) : (w2 & 0xFFFFu));
      const float g = bf16_to_f32((e & 1) ? (g2 >> 16) : (g2 & 0xFFFFu));
      adamw_update(p[e], mo[e], vo[e], g, oc);
    }
#pragma unroll
    for (int e = 0; e < 4; ++e)
      wout[e] = pack_bf16x2(p[2 * e], p[2 * e + 1]);
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      *reinterpret_cast<float4*>(st.m + o + 4 * h) = make_float4(mo[4 * h], mo[4 * h + 1], mo[4 * h + 2], mo[4 * h + 3]);
      *reinterpret_cast<float4*>(st.v + o + 4 * h) = make_float4(vo[4 * h], vo[4 * h + 1], vo[4 * h + 2], vo[4 * h + 3]);
      if (st.master)
        *reinterpret_cast<float4*>(st.master + o + 4 * h) = make_float4(p[4 * h], p[4 * h + 1], p[4 * h + 2], p[4 * h + 3]);
    }
    *reinterpret_cast<i32x4_t*>(st.W + row * st.ldw + col) = i32x4_t{(int)wout[0], (int)wout[1], (int)wout[2], (int)wout[3]};
  }
}

// KD: per valid token, the values of a slab's tiles (KD_STATS) merged, after those of the slabs before (run:
// one row of values per token, written unless this is the last slab), and behind the last slab turned into
// both log-sum-exps and the loss l = lse_s - sum_v p_t(v) zs(v); terms (compact order) feed the mean / sum,
// per_token (row order) is the "none" output. So the values of one slab's tiles are held at a time, 20 bytes
// per 256 ids and token. A workgroup of 16 waves serves 16 tokens: a wave's four groups of 16 lanes fold every
// 64th tile (64-byte reads along the tokens), then the groups and the waves are merged in a fixed order. (One
// thread per token and a serial fold left most CUs idle: 4096 tokens, 501 tiles: 417 us, now 20 in one slab and
// 50 in five.)
constexpr int kKdTok = 16;

__global__ __launch_bounds__(1024) void k_kd_combine(const float* __restrict__ part, int tiles, int64_t ldp,
                                                     float* __restrict__ run, int first, int last,
                                                     const int* __restrict__ idx, const int* __restrict__ nv_ptr,
                                                     float* __restrict__ lse_s, float* __restrict__ lse_t,
                                                     float* __restrict__ terms, float* __restrict__ per_token) {
  __shared__ float red[kKdVals][16][kKdTok];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, t = lane & 15;
  const int i = blockIdx.x * kKdTok + t, nv = *nv_ptr;
  if ((int)blockIdx.x * kKdTok >= nv) return;
  float mt = -INFINITY, st = 0.f, q = 0.f, ms = -INFINITY, ss = 0.f;
  if (!first && wave == 0 && lane < kKdTok && i < nv) {
    mt = run[i];
    st = run[ldp + i];
    q = run[2 * ldp + i];
    ms = run[3 * ldp + i];
    ss = run[4 * ldp + i];
  }
  if (i < nv)
    for (int k = 4 * wave + (lane >> 4); k < tiles; k += 64) {
      const float* p = part + (int64_t)k * kKdVals * ldp + i;
      merge_weighted(mt, st, q, p[0], p[ldp], p[2 * ldp]);
      merge_pair(ms, ss, p[3 * ldp], p[4 * ldp]);
    }
  for (int o = 16; o <= 32; o <<= 1) {
    merge_weighted(mt, st, q, __shfl_xor(mt, o), __shfl_xor(st, o), __shfl_xor(q, o));
    merge_pair(ms, ss, __shfl_xor(ms, o), __shfl_xor(ss, o));
  }
  if (lane < kKdTok) {
    red[0][wave][t] = mt;
    red[1][wave][t] = st;
    red[2][wave][t] = q;
    red[3][wave][t] = ms;
    red[4][wave][t] = ss;
  }
  __syncthreads();
  if (threadIdx.x >= kKdTok || i >= nv) return;
  for (int w = 1; w < 16; ++w) {
    merge_weighted(mt, st, q, red[0][w][t], red[1][w][t], red[2][w][t]);
    merge_pair(ms, ss, red[3][w][t], red[4][w][t]);
  }
  if (!last) {   // (the thread that reads a token's running values is the one that writes them)
    run[i] = mt;
    run[ldp + i] = st;
    run[2 * ldp + i] = q;
    run[3 * ldp + i] = ms;
    run[4 * ldp + i] = ss;
    return;
  }
  const int row = idx[i];
  const float ls = (ms + log2f(ss)) * kLn2;
  lse_s[row] = ls;
  lse_t[row] = (mt + log2f(st)) * kLn2;
  terms[i] = ls - q / st;
  if (per_token) per_token[row] = ls - q / st;
}

// ---------------------------------------------------------------------------------------------
// Host side: validation, plan, workspace carve-up, launches, optional timing.
// ---------------------------------------------------------------------------------------------
enum KernelId { K_COMPACT = 0, K_FWD_STATS, K_COMBINE, K_LOSS, K_GATHER_H, K_BWD_G,
                K_BWD_DW, K_BWD_DH, K_BWD_DHDW, K_DH_FINAL, K_ADAMW, K_SHARD_COMBINE,
                K_KD_Z, K_KD_STATS, K_KD_COMBINE, K_KD_P, K_MISC, K_COUNT };
const char* const kKernelNames[K_COUNT] = {"compact", "fwd_stats", "combine", "loss", "gather_h", "bwd_g",
                                           "bwd_dw", "bwd_dh", "bwd_dhdw", "dh_finalize", "adamw", "shard_combine",
                                           "kd_teacher_z", "kd_student_stats", "kd_combine", "kd_teacher_p", "misc"};

struct Timing {
  std::mutex mu;
  bool on = false;
  static constexpr int kPool = 8192;
  std::vector<hipEvent_t> ev;   // 2 per record
  std::vector<int> kind;
  int used = 0;
};
Timing g_timing;

struct Plan {
  int64_t n, d, v, ldh, ldw, npad;
  int nt_max, vt_count, vt_count3;           // vt_count3: 384-id tiles
  int64_t vc, nslab;
  int64_t gw;                                // 384-id tiles of the forward's vocabulary groups
  int64_t rule_vc;                           // the slab rule's width (many tokens)
  int slab_elem;                             // bytes per id and token that few_token_slab keeps within its budget
  int64_t rows_g;                            // rows of G and dH32: Npad rounded up to a 384-row tile
  // workspace offsets; idx, pos, Nv and the gathered rows Hv form a prefix both passes share
  size_t o_idx, o_pos, o_nv, o_hv, o_pm, o_ps, o_terms, fwd_bytes;
  size_t o_g, o_dh32, o_dh32b, bwd_bytes;    // o_dh32b: accumulator of the second K part (or 0)
  int dh_kz;                                 // most K parts a dH launch takes (1 to 8)
  int part_rows;                             // partial rows of the forward statistics
  bool one_launch;                           // the forward statistics run as one launch
  int fgw;                                   // 384-id tiles of a group of the forward (more than one launch)
  bool split;                                // the forward may cut its last tiles (two partial rows each)
};

inline int64_t round_up(int64_t x, int64_t m) { return (x + m - 1) / m * m; }

// Width, in tiles of tile_rows W rows, of the vocabulary groups the forward and G launches take
// in turn (each group by all token tiles): `tiles` split into equal groups whose W rows fit
// kGroupBytes, so that a group stays in the 256 MB MALL while the token tiles pass.
constexpr int64_t kGroupBytes = (int64_t)160 << 20;
inline int group_tiles(int64_t tiles, int64_t tile_rows, int64_t d) {
  const int64_t bytes = tiles * tile_rows * d * 2;
  const int64_t groups = std::max<int64_t>(1, (bytes + kGroupBytes - 1) / kGroupBytes);
  return (int)std::max<int64_t>(1, (tiles + groups - 1) / groups);
}

// Workgroup rounds of the dW launches over the whole vocabulary with slabs of r 384-id row tiles:
// a slab's ceil(vs / 384) x ceil(D / 256) tiles are cut evenly over the 8 XCDs of 32 CUs each.
int64_t dw_rounds(int64_t v, int64_t d, int64_t r) {
  const int64_t dt = (d + 255) / 256, vt = (v + 383) / 384;
  int64_t total = 0;
  for (int64_t t0 = 0; t0 < vt; t0 += r) {
    const int64_t tiles = std::min(r, vt - t0) * dt;
    total += ((tiles + 7) / 8 + 31) / 32;
  }
  return total;
}

// The slab width, among multiples of 768 ids from max(8192, 4 D) up to what the MALL rule allows
// (the slab's W rows within kGroupBytes, at most 24576 ids), that gives the dW launches the fewest
// workgroup rounds; vc (the rule's own width) unless another needs strictly fewer, and of those
// the widest. A head whose column tiles do not divide 256 (3584 wide: 14) leaves most of a last
// round idle in every slab at the rule's width.
int64_t whole_round_slab(int64_t v, int64_t d, int64_t vc) {
  const int64_t lo = std::max<int64_t>(8192, 4 * d);
  const int64_t hi = std::min(round_up(v, 768), std::max<int64_t>(vc, std::min<int64_t>(24576, kGroupBytes / (2 * d))));
  const int64_t c0 = dw_rounds(v, d, vc / 384);
  int64_t best = vc / 384, cost = c0;
  for (int64_t r = (lo + 767) / 768 * 2; r * 384 <= hi; r += 2) {
    const int64_t c = dw_rounds(v, d, r);
    if (c < cost || (c == cost && c < c0)) {   // r grows: of equal counts the widest
      best = r;
      cost = c;
    }
  }
  return best * 384;
}

// Few tokens: at the width vc chosen above a slab's G launch is then only a few workgroup rounds, of
// which the last, partial one costs most of a round, and every slab pays its launches and a pass over
// the fp32 dH accumulators. When a slab has at most 1024 tiles of 384 ids x 256 tokens (4 rounds of 256
// CUs), the vocabulary is cut into as few equal slabs as keep G within kFewTokenG, whatever V: one
// where [N, V] itself is that small, 1792 tokens of a 128256-id vocabulary. Measured, the rule's slabs, these,
// and as few as 1280 MiB allow (a matrix as large as the bf16 logits; us per step and backward workspace):
//   2048 x 4096 x 128256:        5490 us  313 MiB, 5200 us  516 MiB, 5180 us  796 MiB;
//   1948 x 3584 x 152064:        5515 us  326 MiB, 5225 us  569 MiB, 5150 us  903 MiB;
//   4096 x 4096 x 128256:       10060 us  379 MiB, 9900 us  577 MiB, 9800 us 1263 MiB;
//   4096 x 2048 x 128256:        5270 us  412 MiB, 5295 us  561 MiB, 5185 us 1247 MiB;
//   2048 x (4096 -> 2048) x 128256: 7000 us  318 MiB, 6290 us  693 MiB, 5810 us 1734 MiB;
//   4096 x (4096 -> 2048) x 128256: 12600 us  537 MiB, 11900 us  864 MiB, 11140 us 1774 MiB.
// Above 1024 tiles a partial round is a small share (8192 x 2048 x 128256: 8 rounds) and the memory
// stays with the rule.
// The distillation calls, whose teacher values take 4 bytes per slab id and token, keep those within
// the same bytes.
constexpr int64_t kFewTokenTiles = 1024;
constexpr int64_t kFewTokenG = (int64_t)512 << 20;
int64_t few_token_slab(int64_t v, int64_t npad, int64_t vc, int64_t elem_bytes) {
  if (vc / 384 * (npad / TILE) > kFewTokenTiles) return vc;
  int64_t cap = kFewTokenG / (elem_bytes * round_up(npad, 384)) / 768 * 768;
  cap = std::min<int64_t>(cap, 0x7FFFFFFF / (2 * TILE) / 768 * 768);   // G offsets within a token tile
  if (cap <= vc) return vc;
  const int64_t slabs = (v + cap - 1) / cap;
  return round_up((v + slabs - 1) / slabs, 768);
}

// The forward's launches and its regions after the prefix: the partial rows (pairs per 384-id tile and
// token) and the per-row terms. One launch where a row per tile takes at most 2 D bytes per token or, for
// narrow heads, 4 KiB (512 tiles, 196608 ids: 16384 x 72 x 100000 in five launches of 64 tiles, each waiting
// for the fold of the one before, 1314 us, in one 563); otherwise groups of the slab rule's width, a launch
// each, in two sets of rows and a running pair (as wide as a call of few tokens' slab, the rows would grow
// with V and a group's W rows leave the MALL: 4096 x 2048 x 400000 forward 5450 us, so 4920). A launch of up
// to twice kSplitTiles tiles of all N tokens (fewer may be valid) may cut its last tiles: a second set of
// rows, at most 8 MiB.
//
// least: the form in the least space, which needs no more than any version of this library has asked for: no
// cut tiles, and where there may be more rows than before (narrow heads, and widths that are not a multiple
// of 64, which once took at most 64) groups of 24 tiles, 2 x 24 + 1 rows.
void plan_forward(Plan* pl, bool least) {
  const int64_t vt = pl->vt_count3, tiles = vt * pl->nt_max;
  const bool few = least && (pl->d % KSLICE != 0 || vt > pl->d / 4);
  pl->one_launch = (few ? vt <= 24 : vt <= std::max<int64_t>(pl->d / 4, 512)) && tiles <= INT32_MAX;
  pl->split = !least && pl->one_launch && tiles <= 2 * kSplitTiles;
  pl->fgw = few ? 24 : (int)(pl->rule_vc / 384);
  const int64_t rows = pl->one_launch || vt <= pl->fgw ? vt : 2 * (int64_t)pl->fgw + 1;
  // (not below two rows per 256 ids, up to 64: small heads then ask for the same bytes in either form)
  pl->part_rows = (int)std::max<int64_t>(pl->split ? 2 * rows : rows, few ? 0 : 2 * std::min(pl->vt_count, 32));
  const size_t arr = (4 * (size_t)pl->part_rows * pl->npad + 255) / 256 * 256;
  pl->o_pm = pl->o_hv + (2 * (size_t)pl->d * pl->npad + 255) / 256 * 256;
  pl->o_ps = pl->o_pm + arr;
  pl->o_terms = pl->o_ps + arr;
  pl->fwd_bytes = pl->o_terms + 4 * (size_t)pl->npad;
}

// The plan of a forward in workspace_bytes. The form follows from the problem alone wherever the workspace
// holds the size that is reported for it, so that its size never shows in the results; a smaller one, which
// callers may hold from before the present forms, is served in the least form as long as that fits.
bool forward_fits(Plan* pl, size_t workspace_bytes) {
  if (pl->fwd_bytes > workspace_bytes) plan_forward(pl, true);
  return pl->fwd_bytes <= workspace_bytes;
}

// The backward's slabs, its dH launches and its regions after the prefix.
//
// least: the form in the least space, which needs no more than any version of this library has asked for: the
// rule's slabs, and as many K parts as fill the CUs once with the tiles of all N tokens.
void plan_backward(Plan* pl, bool least) {
  const int64_t vround = round_up(pl->v, 768);
  pl->vc = pl->rule_vc;
  if (pl->vc < vround) pl->vc = few_token_slab(pl->v, pl->npad, pl->vc, pl->slab_elem);
  if (least) pl->vc = std::min(pl->vc, pl->rule_vc);   // (as many equal slabs as the rule's may be narrower)
  pl->nslab = (pl->v + pl->vc - 1) / pl->vc;
  auto take = [](size_t& cur, size_t bytes) { size_t o = cur; cur += (bytes + 255) / 256 * 256; return o; };
  size_t cur = pl->o_hv;
  take(cur, 2 * (size_t)pl->d * pl->npad);
  // G and the fp32 dH accumulators hold every row a 384-row dH tile can address (the tiles of
  // the last token rows reach past Npad), so that no access leaves its region
  pl->rows_g = round_up(pl->npad, 384);
  pl->o_g = take(cur, 2 * (size_t)pl->rows_g * pl->vc);
  // dH launches with fewer 384 x 256 output tiles than the 256 CUs split K into parts (at most 8), each
  // accumulated in an accumulator of its own; the kernel takes as many as the live tiles (of Nv, not N,
  // tokens) leave CUs for, so twice as many are reserved as the tiles of all N tokens would take
  const int64_t dh_tiles = (pl->npad + 383) / 384 * ((pl->d + TILE - 1) / TILE), units = least ? 256 : 512;
  pl->dh_kz = dh_tiles >= 256 ? 1 : (int)std::min<int64_t>(8, (units + dh_tiles - 1) / dh_tiles);
  const size_t part = 4 * (size_t)pl->rows_g * pl->d;     // a multiple of 256 bytes
  pl->o_dh32 = take(cur, part * pl->dh_kz);
  pl->o_dh32b = pl->dh_kz > 1 ? pl->o_dh32 + part : 0;
  pl->bwd_bytes = cur;
}

lce_status_t make_plan(const lce_problem_t* p, Plan* pl, bool wide_slabs = true) {
  if (!p) return LCE_ERR_NULL;
  if ((p->flags & ~(LCE_FLAG_ACCUMULATE_DW | LCE_FLAG_REUSE_FORWARD)) != 0) return LCE_ERR_ARG;
  if (p->n < 0 || p->d < 1 || p->v < 1) return LCE_ERR_SHAPE;
  if (p->d % 8 != 0) return LCE_ERR_UNSUPPORTED;
  if (p->reduction != LCE_REDUCE_MEAN && p->reduction != LCE_REDUCE_SUM && p->reduction != LCE_REDUCE_NONE)
    return LCE_ERR_UNSUPPORTED;
  if (p->target_bytes != 4 && p->target_bytes != 8) return LCE_ERR_UNSUPPORTED;
  const int64_t ldh = p->ld_h ? p->ld_h : p->d, ldw = p->ld_w ? p->ld_w : p->d;
  if (ldh < p->d || ldw < p->d) return LCE_ERR_SHAPE;
  if (ldh % 8 != 0 || ldw % 8 != 0) return LCE_ERR_ALIGN;
  // 32-bit limits: token / vocabulary indices, and byte offsets inside one buffer resource
  if (p->n >= (int64_t)1 << 30 || p->v >= (int64_t)1 << 30 || p->d >= (int64_t)1 << 20) return LCE_ERR_SHAPE;
  if ((uint64_t)p->n * ldh * 2 > 0x7FFFFFFFull) return LCE_ERR_SHAPE;
  // byte offsets within one 384-row tile of W (bf16) and of the fp32 optimizer state
  if ((uint64_t)384 * ldw * 2 > 0x7FFFFFFFull || (uint64_t)384 * p->d * 4 > 0x7FFFFFFFull) return LCE_ERR_SHAPE;
  pl->n = p->n; pl->d = p->d; pl->v = p->v; pl->ldh = ldh; pl->ldw = ldw;
  pl->npad = round_up(p->n > 0 ? p->n : 1, TILE);
  pl->nt_max = (int)(pl->npad / TILE);
  pl->vt_count = (int)((p->v + TILE - 1) / TILE);
  pl->vt_count3 = (int)((p->v + 383) / 384);
  // backward vocabulary slab: about 4 D columns (at least 8192) keeps G at O(N D) while halving
  // the dH accumulator passes of a 2 D slab. Narrower heads take up to 24576 ids while the slab's
  // W rows fit kGroupBytes (they stay in the MALL while G's token tiles pass), which cuts their
  // fp32 accumulator passes further (the distillation calls keep the narrow slab: their teacher
  // probabilities take 4 bytes per slab id and token). A multiple of 16 tiles of 384 ids, so that
  // the dW launch of a 4096-wide head is whole rounds of workgroups on 256 CUs; for other widths
  // whole_round_slab picks the width whose dW launches leave the fewest idle CUs. Calls of few
  // tokens take wider slabs, within a fixed number of bytes (few_token_slab).
  int64_t vc = 4 * p->d;
  if (wide_slabs) vc = std::max<int64_t>(vc, std::min<int64_t>(24576, kGroupBytes / (2 * p->d) / 6144 * 6144));
  if (vc < 8192) vc = 8192;
  vc = round_up(vc, 16 * 384);
  // a multiple of 768 in any case: both 256- and 384-wide G tiles end inside a G row
  const int64_t vround = round_up(p->v, 768);
  if (vc > vround) vc = vround;
  // the forward's groups keep the rule's width (they only order its tiles; a wider group's W rows
  // leave the MALL)
  pl->gw = vc / 384;
  if (wide_slabs && vc < vround) vc = whole_round_slab(p->v, p->d, vc);
  pl->rule_vc = vc;
  pl->slab_elem = wide_slabs ? 2 : 4;
  if ((uint64_t)TILE * pl->npad * 2 > 0x7FFFFFFFull || (uint64_t)TILE * vc * 2 > 0x7FFFFFFFull) return LCE_ERR_SHAPE;

  auto take = [](size_t& cur, size_t bytes) { size_t o = cur; cur += (bytes + 255) / 256 * 256; return o; };
  size_t cur = 0;
  pl->o_idx = take(cur, 4 * (size_t)pl->npad);
  pl->o_pos = take(cur, 4 * (size_t)pl->npad);
  pl->o_nv = take(cur, 256);
  // valid rows of H, gathered by the forward and by the backward; a backward with
  // LCE_FLAG_REUSE_FORWARD finds the forward's here
  pl->o_hv = take(cur, 2 * (size_t)p->d * pl->npad);
  // a forward beyond the library's fixed array takes the least form if that fits it, so that
  // lce_forward_noalloc and lce_forward run the same launches for every problem the former serves
  plan_forward(pl, false);
  if (pl->fwd_bytes > (size_t)LCE_NOALLOC_SCRATCH_BYTES) {
    plan_forward(pl, true);
    if (pl->fwd_bytes > (size_t)LCE_NOALLOC_SCRATCH_BYTES) plan_forward(pl, false);
  }
  plan_backward(pl, false);
  return LCE_OK;
}

inline bool aligned16(const void* p) { return ((uintptr_t)p & 15) == 0; }

lce_status_t make_adamw(const lce_adamw_t* o, AdamWConst* c) {
  if (!o) return LCE_ERR_NULL;
  if (o->reserved != 0 || o->step < 1) return LCE_ERR_ARG;
  if (!(o->lr >= 0.f && o->lr < INFINITY) || !(o->beta1 >= 0.f && o->beta1 < 1.f) ||
      !(o->beta2 >= 0.f && o->beta2 < 1.f) || !(o->eps >= 0.f && o->eps < INFINITY) ||
      !(o->weight_decay >= 0.f && o->weight_decay < INFINITY))
    return LCE_ERR_ARG;
  const double lr = o->lr, b1 = o->beta1, b2 = o->beta2;
  c->keep = (float)(1.0 - lr * (double)o->weight_decay);
  c->beta1 = o->beta1;
  c->omb1 = (float)(1.0 - b1);
  c->beta2 = o->beta2;
  c->omb2 = (float)(1.0 - b2);
  c->step_size = (float)(lr / (1.0 - pow(b1, (double)o->step)));
  c->inv_sqrt_bc2 = (float)(1.0 / sqrt(1.0 - pow(b2, (double)o->step)));
  c->eps = o->eps;
  return LCE_OK;
}

unsigned adamw_grid(int64_t v, int64_t d) {
  const int64_t chunks = v * (d / 8);
  const int64_t blocks = (chunks + 255) / 256;
  return (unsigned)(blocks < 16384 ? blocks : 16384);
}

// k_combine with 64 tokens a workgroup: enough workgroups all the same, and dot products so short that four side by
// side fill a wave's loads. 64 tokens against 16: 32768 tokens of 256 / 1024 / 2048 x 5000 ids 14 / 22 / 34 us
// against 21 / 25 / 36, x 32768 17 / 26 / 44 against 23 / 29 / 46, x 128256 28 / 47 / 73 against 37 / 47 / 73; but
// 16384 tokens of 256 / 1024 / 2048 x 128256 24 / 36 / 49 against 20 / 29 / 37, and fewer tokens more so.
inline bool wide_combine(const Plan& pl) { return pl.n > 16384 && pl.d <= 1536; }

struct Launcher {
  hipStream_t s;
  lce_status_t st = LCE_OK;
  // the kernel's arguments, converted to its parameter types, passed by address
  template <typename... KArgs>
  hipError_t launch(void (*kern)(KArgs...), dim3 grid, dim3 block, KArgs... a) {
    void* ptrs[sizeof...(KArgs) + 1] = {static_cast<void*>(&a)..., nullptr};
    return hipLaunchKernel(reinterpret_cast<const void*>(kern), grid, block, ptrs, 0, s);
  }
  template <typename... KArgs, typename... Args>
  void operator()(int kind, void (*kern)(KArgs...), dim3 grid, dim3 block, Args... args) {
    if (st != LCE_OK) return;
    if (grid.x == 0 || grid.y == 0 || grid.z == 0) return;
    int slot = -1;
    if (g_timing.on) {
      std::lock_guard<std::mutex> lk(g_timing.mu);
      if (g_timing.on && g_timing.used < Timing::kPool) {
        slot = g_timing.used++;
        g_timing.kind[slot] = kind;
      }
    }
    if (slot >= 0 && hipEventRecord(g_timing.ev[2 * slot], s) != hipSuccess) { st = LCE_ERR_HIP; return; }
    // the launch's own status, without reading (and clearing) the thread's last-error slot, which
    // may hold an earlier, unrelated call's error
    if (launch(kern, grid, block, static_cast<KArgs>(args)...) != hipSuccess) {
      st = LCE_ERR_HIP;
      return;
    }
    if (slot >= 0 && hipEventRecord(g_timing.ev[2 * slot + 1], s) != hipSuccess) st = LCE_ERR_HIP;
  }
};

// Which part of the vocabulary W holds: ids [v_begin, v_begin + p->v) of v_total (the whole
// vocabulary: v_begin = 0, v_total = p->v).
struct ShardInfo {
  int64_t v_total, v_begin;
};

lce_status_t shard_info(const lce_problem_t* p, const lce_shard_t* sh, ShardInfo* si) {
  if (!p || !sh) return LCE_ERR_NULL;
  if (sh->v_total < 1 || sh->v_total >= (int64_t)1 << 30 || sh->v_begin < 0 || p->v < 1 ||
      sh->v_begin + p->v > sh->v_total)
    return LCE_ERR_SHAPE;
  si->v_total = sh->v_total;
  si->v_begin = sh->v_begin;
  return LCE_OK;
}

// Partial rows that k_combine folds for one head: `count` rows of Npad from (m, s), after an
// optional running pair (run_m, run_s).
struct PartRows {
  const float* m;
  const float* s;
  int count;          // tiles; two rows each where the launch was split (k_fwd_tile)
  int split;
  const float* run_m;
  const float* run_s;
};

// The valid rows of H (row stride ldh, d wide) made contiguous in hv.
void launch_gather(Launcher& L, const uint16_t* H, int64_t ldh, int d, int64_t npad, const int* idx, const int* nv,
                   uint16_t* hv) {
  L(K_GATHER_H, k_gather_rows, dim3((unsigned)std::min<int64_t>((npad * (d / 8) + 255) / 256, 16384)), dim3(256), H,
    ldh, idx, nv, d, hv);
}

// Vocabulary statistics, in log2 units of the logits: the valid rows of H are gathered into hv and the
// tiles run, in one launch or one per group of tiles (as the plan that sized the partial rows decides).
PartRows launch_fwd_stats(Launcher& L, const Plan& layout, const uint16_t* W, int64_t ldw, const uint16_t* H,
                          int64_t ldh, const int* idx, const int* nv, uint16_t* hv, float* pm, float* ps) {
  const int v = (int)layout.v, npad = (int)layout.npad, nt_max = layout.nt_max, d = (int)layout.d;
  const auto kernel = d % KSLICE == 0 ? k_fwd_tile<false> : k_fwd_tile<true>;
  launch_gather(L, H, ldh, d, npad, idx, nv, hv);
  const int gw = layout.fgw;
  const int ntl = layout.vt_count3;
  if (layout.one_launch) {
    // one launch: the groups only order the tiles (as wide as the slab rule's width, or narrower
    // where its W rows would not stay in the MALL)
    const TileOrder to = tile_order(ntl, nt_max, group_tiles(layout.gw, Geo<3>::TM, d), layout.split);
    L(K_FWD_STATS, kernel, dim3(to.grid), dim3(Geo<3>::NT), W, ldw, v, (const uint16_t*)hv,
      (int64_t)d, nv, d, 0, ntl, to.gw, (int)layout.split, pm, ps, (const float*)nullptr, (const float*)nullptr, 0,
      (float*)nullptr, (float*)nullptr, 0, npad, kLog2e);
    return PartRows{pm, ps, ntl, layout.split, nullptr, nullptr};
  }
  // one group per launch; row sets: parity 0 at rows [0, gw), parity 1 at [gw, 2 gw), the
  // running pair at row 2 gw
  const int ng = (ntl + gw - 1) / gw;
  const int64_t rs = (int64_t)gw * npad;
  float* run_m = pm + 2 * rs;
  float* run_s = ps + 2 * rs;
  for (int g = 0; g < ng; ++g) {
    const int tm0 = g * gw, wl = std::min(gw, ntl - tm0);
    const int64_t cur = (g & 1) * rs, prev = ((g + 1) & 1) * rs;
    const TileOrder to = tile_order(wl, nt_max, wl);
    L(K_FWD_STATS, kernel, dim3(to.grid), dim3(Geo<3>::NT), W, ldw, v, (const uint16_t*)hv,
      (int64_t)d, nv, d, tm0, wl, to.gw, 0, pm + cur, ps + cur,
      g > 0 ? (const float*)(pm + prev) : (const float*)nullptr, (const float*)(ps + prev), gw, run_m, run_s,
      g == 1 ? 1 : 0, npad, kLog2e);
  }
  const int64_t last = ((ng - 1) & 1) * rs;
  return PartRows{pm + last, ps + last, ntl - (ng - 1) * gw, 0, ng > 1 ? run_m : nullptr, run_s};
}

// The forward pass behind lce_forward and (tgt_part != null) lce_forward_shard.
lce_status_t forward_impl(const lce_problem_t* p, const ShardInfo* shard, const void* H, const void* W,
                          const void* targets, float* loss, float* lse, float* tgt_part, int32_t* n_valid,
                          int32_t* dev_status, void* workspace, size_t workspace_bytes, void* stream) {
  Plan pl;
  lce_status_t st = make_plan(p, &pl);
  if (st != LCE_OK) return st;
  const ShardInfo si = shard ? *shard : ShardInfo{pl.v, 0};
  if ((!shard && !loss) || (shard && !tgt_part) || !n_valid) return LCE_ERR_NULL;
  if (pl.n > 0 && (!H || !W || !targets || !lse || !workspace)) return LCE_ERR_NULL;
  if (pl.n > 0 && (!aligned16(H) || !aligned16(W) || ((uintptr_t)workspace & 255) != 0)) return LCE_ERR_ALIGN;
  if (pl.n > 0 && !forward_fits(&pl, workspace_bytes)) return LCE_ERR_WORKSPACE;
  Launcher L{(hipStream_t)stream};
  const bool none = !shard && p->reduction == LCE_REDUCE_NONE;
  if (pl.n == 0) {
    L(K_MISC, k_fwd_empty, dim3(1), dim3(64), (none || shard) ? (float*)nullptr : loss, n_valid, dev_status);
    return L.st;
  }
  char* ws = (char*)workspace;
  int* idx = (int*)(ws + pl.o_idx);
  int* pos = (int*)(ws + pl.o_pos);
  int* nv = (int*)(ws + pl.o_nv);
  float* pm = (float*)(ws + pl.o_pm);
  float* ps = (float*)(ws + pl.o_ps);
  float* terms = (float*)(ws + pl.o_terms);
  const uint16_t* h = (const uint16_t*)H;
  const uint16_t* w = (const uint16_t*)W;

  // rows that are not valid get lse 0 and a zero per-token loss (or shard target logit)
  L(K_COMPACT, k_compact, dim3(1), dim3(1024), targets, p->target_bytes, pl.n, si.v_total, p->ignore_index,
    idx, pos, nv, n_valid, dev_status, lse, none ? loss : tgt_part, (float*)nullptr);
  const PartRows pr = launch_fwd_stats(L, pl, w, pl.ldw, h, pl.ldh, (const int*)idx, (const int*)nv,
                                       (uint16_t*)(ws + pl.o_hv), pm, ps);
  const int ctok = wide_combine(pl) ? 64 : 16;
  L(K_COMBINE, ctok == 64 ? k_combine<64> : k_combine<16>, dim3((unsigned)((pl.n + ctok - 1) / ctok)), dim3(1024), h,
    pl.ldh, w, pl.ldw, targets, p->target_bytes, si.v_begin, pl.v, (const int*)idx, (const int*)nv, (int)pl.d,
    pr.count, pr.split, pr.m, pr.s, (int)pl.npad, pr.run_m, pr.run_s, lse, terms, none ? loss : (float*)nullptr,
    tgt_part);
  if (!none && !shard) L(K_LOSS, k_loss, dim3(1), dim3(1024), (const float*)terms, (const int*)nv, p->reduction, loss);
  return L.st;
}

// Teacher head of the distillation loss, as the student's backward needs it: the teacher's
// probabilities are recomputed slab by slab into an fp32 buffer P [Vc][Npad] placed after the
// student's backward workspace.
struct KdArgs {
  const uint16_t* ht;
  int64_t ldht;
  const uint16_t* wt;
  int64_t ldwt;
  int dt;
  const float* lse_t;
  float scale2, inv_t;
  bool formed;   // the valid-row list and the teacher's gathered rows are in place (fused KD call)
};

// The teacher's pass over one slab: its logits (Z_WRITE) or probabilities (P_WRITE, from lse_t) into P
// [Vc][Npad], on 12-wave tiles over the gathered rows hvt, or (null) 8-wave tiles that gather.
template <int kMode>
void launch_teacher(Launcher& L, int kind, const KdArgs& kd, const uint16_t* hvt, const Plan& pl, int64_t v0, int vs,
                    const int* idx, const int* nv, float* P) {
  const int wm = hvt ? 3 : 2, rows = 128 * wm, tm = (vs + rows - 1) / rows;
  const TileOrder to = tile_order(tm, pl.nt_max, hvt ? group_tiles(tm, rows, kd.dt) : tm);
  L(kind, hvt ? k_kd_tile<kMode, 3> : k_kd_tile<kMode, 2>, dim3(to.grid), dim3(256 * wm), kd.wt, kd.ldwt, v0, vs,
    hvt ? hvt : kd.ht, hvt ? (int64_t)kd.dt : kd.ldht, pl.n, idx, nv, kd.lse_t,
    (const float*)nullptr, (const int*)nullptr, (int)LCE_REDUCE_MEAN, kd.dt, tm, (uint16_t*)nullptr, (int)pl.vc,
    (int)pl.npad, kd.scale2, kd.inv_t, P, (float*)nullptr, to.gw);
}

inline size_t kd_p_bytes(const Plan& pl) { return (size_t)4 * pl.vc * pl.npad; }

// Id tiles per vocabulary group of the student's launches: half the W rows of an LCE group, since the
// teacher's values of every tile stream through the MALL beside them. (A wide slab as one group lost its W
// rows between token tiles: 3072 valid tokens, 2048 wide, 64512 ids: statistics 1790 us and G 1980, in groups
// of 160 MiB 1625 and 1700, of 80 MiB 1567 and 1675, of 40 MiB 1582 and 1684.)
inline int student_group(int tiles, int64_t d) { return group_tiles(tiles, TILE, 2 * d); }

// The teacher's valid rows gathered for its 12-wave probability pass (Npad x Dt bf16), when
// Dt % 64 == 0; placed after P.
inline size_t kd_hvt_bytes(const Plan& pl, int64_t dt) {
  return dt % KSLICE == 0 ? ((size_t)2 * dt * pl.npad + 255) / 256 * 256 : 0;
}

// The backward pass behind lce_backward (dW != null), lce_backward_adamw (adamw != null),
// lce_backward_shard (shard != null, fp32 dH term in dHf) and lce_kd_backward (kd != null). `want` says
// which gradients a caller uses (lce_backward_select): the contraction of the other is not run, a
// quarter of the pass's work (the frozen head of 4096 x 4096 x 128256: step 9750 -> 7470 us).
enum Want { WANT_DH = 1, WANT_DW = 2 };
lce_status_t backward_impl(const lce_problem_t* p, const ShardInfo* shard, const void* H, const void* W,
                           const void* targets, const float* lse, const int32_t* n_valid, const float* grad_loss,
                           void* dH, float* dHf, uint16_t* dW, const AdamWState* adamw, const AdamWConst* oc,
                           void* workspace, size_t workspace_bytes, void* stream, const KdArgs* kd = nullptr,
                           int want = WANT_DH | WANT_DW) {
  Plan pl;
  // the distillation calls keep the narrow slab of their own plan (make_kd_plan)
  lce_status_t st = make_plan(p, &pl, kd == nullptr);
  if (st != LCE_OK) return st;
  const ShardInfo si = shard ? *shard : ShardInfo{pl.v, 0};
  void* dH_any = dHf ? (void*)dHf : dH;
  if (!W || !grad_loss || (!n_valid && p->reduction == LCE_REDUCE_MEAN)) return LCE_ERR_NULL;
  if (pl.n > 0 && (!H || !targets || !lse || (!dH_any && (want & WANT_DH)) || !workspace)) return LCE_ERR_NULL;
  if (!aligned16(W)) return LCE_ERR_ALIGN;
  if (pl.n > 0 && (!aligned16(H) || !aligned16(dH_any) || ((uintptr_t)workspace & 255) != 0)) return LCE_ERR_ALIGN;
  // (a workspace smaller than what is reported, as callers may hold from before the present slabs, is served in
  // the least form)
  auto need = [&] { return pl.bwd_bytes + (kd ? kd_p_bytes(pl) + kd_hvt_bytes(pl, kd->dt) : 0); };
  if (pl.n > 0 && workspace_bytes < need()) {
    plan_backward(&pl, true);
    if (workspace_bytes < need()) return LCE_ERR_WORKSPACE;
  }
  const bool accumulate = (p->flags & LCE_FLAG_ACCUMULATE_DW) != 0;
  const AdamWState as = adamw ? *adamw : AdamWState{nullptr, 0, nullptr, nullptr, nullptr};
  const AdamWConst c = oc ? *oc : AdamWConst{};
  Launcher L{(hipStream_t)stream};
  if (pl.n == 0) {
    // no tokens: dW is zero, so the fused step is a step with a zero gradient
    if (adamw) {
      L(K_ADAMW, k_adamw, dim3(adamw_grid(pl.v, pl.d)), dim3(256), pl.v, (int)pl.d, (const uint16_t*)nullptr, as, c);
    } else if ((want & WANT_DW) && !accumulate) {
      const int64_t n16 = pl.v * pl.d / 8;
      L(K_MISC, k_zero16, dim3((unsigned)((n16 + 255) / 256)), dim3(256), (uint4*)dW, n16);
    }
    return L.st;
  }
  char* ws = (char*)workspace;
  int* idx = (int*)(ws + pl.o_idx);
  int* pos = (int*)(ws + pl.o_pos);
  int* nv = (int*)(ws + pl.o_nv);
  uint16_t* hv = (uint16_t*)(ws + pl.o_hv);
  uint16_t* g = (uint16_t*)(ws + pl.o_g);
  float* dh32 = (float*)(ws + pl.o_dh32);
  float* dh32b = pl.dh_kz > 1 ? (float*)(ws + pl.o_dh32b) : nullptr;   // accumulator of K part 1 (parts follow)
  const uint16_t* h = (const uint16_t*)H;
  const uint16_t* w = (const uint16_t*)W;
  const int d = (int)pl.d, npad = (int)pl.npad, vc = (int)pl.vc;

  // with LCE_FLAG_REUSE_FORWARD the workspace holds the forward's valid-row list and the rows Hv;
  // otherwise both are formed again
  const bool reuse = kd ? kd->formed : (p->flags & LCE_FLAG_REUSE_FORWARD) != 0;
  if (!reuse)
    L(K_COMPACT, k_compact, dim3(1), dim3(1024), targets, p->target_bytes, pl.n, si.v_total, p->ignore_index,
      idx, pos, nv, (int*)nullptr, (int*)nullptr, (float*)nullptr, (float*)nullptr, (float*)nullptr);
  // Hv[i] = H[idx[i]] for i < Nv, zero rows up to round_up(Nv, 64)
  if (kd || !reuse) launch_gather(L, h, pl.ldh, d, npad, idx, nv, hv);
  // KD: the teacher's valid rows for its 12-wave probability pass
  uint16_t* hvt = (kd && kd_hvt_bytes(pl, kd->dt) > 0) ? (uint16_t*)(ws + pl.bwd_bytes + kd_p_bytes(pl)) : nullptr;
  if (hvt && !kd->formed) launch_gather(L, kd->ht, kd->ldht, kd->dt, npad, idx, nv, hvt);
  const int dt = (d + TILE - 1) / TILE;
  const int dh_tiles = (int)((pl.npad + Geo<kDhWM>::TM - 1) / Geo<kDhWM>::TM);
  void (*dw_kernel)(const uint16_t*, int, int, int, const uint16_t*, int, const int*, int, uint16_t*, int64_t,
                    AdamWState, AdamWConst) =
      adamw ? k_bwd_dw<DW_ADAMW, kDwWM> : accumulate ? k_bwd_dw<DW_ACCUMULATE, kDwWM> : k_bwd_dw<DW_STORE, kDwWM>;
  // dH and dW of a slab as one launch (k_bwd_dhdw; not with the optimizer step, whose dW launch updates
  // the W rows that dH reads) up to kMergeTiles dH tiles, 3 rounds of the CUs, of all N tokens. One launch
  // against two, dH + dW: 4096 tokens of a 16032 x 8192 shard (352 tiles) 1706 -> 1283 us; 8192 x 8192 x
  // 64000 (704) 11.5 -> 10.4 ms; 1948 x 3584 x 152064 (84) 2630 -> 2545 us; 256 x 512 x 4096 (2) 48 -> 25 us;
  // 16384 x 4096 x 128256 (688) the same within 1 %; 16384 x 4352 x 100000 (731) 21.0 -> 19.5 ms; 24576 x 3072
  // x 32768 (768) 6050 -> 5580 us, x 128256 the same; narrow heads with many tokens (256 to 1024 wide, 8192 to
  // 32768 tokens, 43 to 344 tiles) 1 to 25 % less; but 32768 x 3584 x 152064 (1204, several dH rounds anyway)
  // 37.9 -> 38.3 ms.
  static_assert(kDhWM == kDwWM, "one launch runs both");
  constexpr int kMergeTiles = 768;
  const bool merge = !adamw && want == (WANT_DH | WANT_DW) && (int64_t)dh_tiles * dt <= kMergeTiles;
  for (int64_t s = 0; s < pl.nslab; ++s) {
    const int64_t v0 = s * pl.vc;
    const int vs = (int)(pl.v - v0 < pl.vc ? pl.v - v0 : pl.vc);
    const int tm = (vs + TILE - 1) / TILE;
    if (kd) {
      // teacher probabilities of this slab, then G = c (softmax(zs / T) - P) / T
      float* P = (float*)(ws + pl.bwd_bytes);
      launch_teacher<P_WRITE>(L, K_KD_P, *kd, hvt, pl, v0, vs, idx, nv, P);
      const TileOrder to = tile_order(tm, pl.nt_max, student_group(tm, pl.d));
      L(K_BWD_G, k_kd_tile<G_SOFT, 2>, dim3(to.grid), dim3(NTHREADS), w, pl.ldw, v0, vs, h,
        pl.ldh, pl.n, (const int*)idx, (const int*)nv, lse, grad_loss,
        (const int*)n_valid, p->reduction, d, tm, g, vc, npad, kd->scale2, kd->inv_t, P, (float*)nullptr, to.gw);
    } else {
      const int tmg = (vs + Geo<3>::TM - 1) / Geo<3>::TM;
      const TileOrder to = tile_order(tmg, pl.nt_max, group_tiles(tmg, Geo<3>::TM, d), true);
      L(K_BWD_G, d % KSLICE == 0 ? k_bwd_g<false> : k_bwd_g<true>, dim3(to.grid), dim3(Geo<3>::NT), w, pl.ldw, v0, vs,
        (const uint16_t*)hv, (int64_t)d, targets, p->target_bytes, si.v_begin, (const int*)idx, (const int*)nv, lse,
        grad_loss, (const int*)n_valid, p->reduction, d, tmg, to.gw, 1, g, vc);
    }
    const unsigned bdh = (unsigned)dh_grid(pl.npad, d, pl.dh_kz);
    const int tmw = (vs + Geo<kDwWM>::TM - 1) / Geo<kDwWM>::TM;
    const unsigned bdw = (unsigned)dw_grid(tmw, d);
    // dH reads the slab's W rows before the dW launch, whose AdamW epilogue (in-backward step)
    // may update them; later slabs read only their own rows
    if (merge) {
      L(K_BWD_DHDW, accumulate ? k_bwd_dhdw<DW_ACCUMULATE, kDwWM> : k_bwd_dhdw<DW_STORE, kDwWM>, dim3(bdh + bdw),
        dim3(Geo<kDwWM>::NT), (const uint16_t*)g, vc, npad, vs, w + v0 * pl.ldw, pl.ldw, pl.v - v0, d, (const int*)nv,
        dh32, (int)(s > 0), pl.dh_kz, dh32b, (int)pl.rows_g, (int)bdh, (const uint16_t*)hv, tmw, dW, v0);
      continue;
    }
    if (want & WANT_DH)
      L(K_BWD_DH, k_bwd_dh<kDhWM>, dim3(bdh), dim3(Geo<kDhWM>::NT), (const uint16_t*)g, vc, vs, w + v0 * pl.ldw, pl.ldw,
        pl.v - v0, d, (const int*)nv, dh32, (int)(s > 0), pl.dh_kz, dh32b, (int)pl.rows_g);
    if (want & WANT_DW)
      L(K_BWD_DW, dw_kernel, dim3(bdw), dim3(Geo<kDwWM>::NT), (const uint16_t*)g, vc, npad, vs, (const uint16_t*)hv, d,
        (const int*)nv, tmw, dW, v0, as, c);
  }
  if (!(want & WANT_DH)) return L.st;
  const int64_t nthr = pl.n * pl.d / 8;
  L(K_DH_FINAL, k_dh_finalize, dim3((unsigned)((nthr + 255) / 256)), dim3(256), (const float*)dh32,
    (int64_t)pl.rows_g * d, pl.dh_kz, (const int*)pos, pl.n, d, (uint16_t*)dH, dHf, 1, (const int*)nv, (int)pl.rows_g);
  return L.st;
}

// ---- knowledge distillation --------------------------------------------------------------------
struct KdPlan {
  lce_problem_t ps, pt;   // student and teacher heads as LCE problems
  Plan s, t;
  float scale2, inv_t;
  // the forward's regions: the student's valid-row list, then the values of a slab's tiles and the running
  // ones, the per-row terms and the teacher's logits and gathered rows. (In the fused call these two lie where
  // the backward keeps its probabilities and gathered rows, the values in G and the terms in the dH
  // accumulators, which the backward writes after the forward has read them.)
  size_t o_q, o_terms, o_p, o_hvt, fwd_bytes, bwd_bytes;
};

lce_status_t make_kd_plan(const lce_kd_problem_t* p, KdPlan* k, bool least = false) {
  if (!p) return LCE_ERR_NULL;
  if (p->reserved != 0) return LCE_ERR_ARG;
  if (!(p->temperature > 0.f && p->temperature < INFINITY)) return LCE_ERR_ARG;
  if (p->flags & LCE_FLAG_REUSE_FORWARD) return LCE_ERR_ARG;   // the KD calls lay out their own workspace
  k->ps = lce_problem_t{p->n, p->ds, p->v, p->ld_hs, p->ld_ws, p->ignore_index, p->reduction, p->target_bytes, p->flags};
  k->pt = lce_problem_t{p->n, p->dt, p->v, p->ld_ht, p->ld_wt, p->ignore_index, p->reduction, p->target_bytes, 0};
  lce_status_t st = make_plan(&k->ps, &k->s, false);
  if (st != LCE_OK) return st;
  st = make_plan(&k->pt, &k->t, false);
  if (st != LCE_OK) return st;
  if (least) plan_backward(&k->s, true);
  k->scale2 = (float)(1.4426950408889634 / (double)p->temperature);
  k->inv_t = (float)(1.0 / (double)p->temperature);
  auto up = [](size_t x) { return (x + 255) / 256 * 256; };
  const size_t q_rows = (std::min(k->s.vc, k->s.v) + TILE - 1) / TILE + (k->s.nslab > 1 ? 1 : 0);
  const size_t q_bytes = up(4 * kKdVals * q_rows * k->s.npad), t_bytes = up(4 * (size_t)k->s.npad);
  const size_t p_bytes = up(kd_p_bytes(k->s)), hvt_bytes = kd_hvt_bytes(k->s, k->t.d);
  size_t cur = up(k->s.o_hv);   // after idx, pos and Nv
  k->o_q = cur;
  k->o_terms = k->o_q + q_bytes;
  k->o_p = k->o_terms + t_bytes;
  k->o_hvt = k->o_p + p_bytes;
  k->fwd_bytes = k->o_hvt + hvt_bytes;
  k->bwd_bytes = k->s.bwd_bytes + kd_p_bytes(k->s) + hvt_bytes;
  return LCE_OK;
}

// The KD forward: both heads' log-sum-exps and the loss. Per slab, one teacher pass (its logits into P)
// and one student pass (KD_STATS), then a merge of its tiles' values.
lce_status_t kd_forward_launches(Launcher& L, const lce_kd_problem_t* p, const KdPlan& k, const KdArgs& kd,
                                 const uint16_t* hs, const uint16_t* wsm, const void* targets, float* loss,
                                 float* lse_s, float* lse_t, int32_t* n_valid, int32_t* dev_status, char* ws,
                                 size_t o_q, size_t o_terms, size_t o_p, size_t o_hvt) {
  const Plan& pl = k.s;
  const bool none = p->reduction == LCE_REDUCE_NONE;
  int* idx = (int*)(ws + pl.o_idx);
  int* nv = (int*)(ws + pl.o_nv);
  float* terms = (float*)(ws + o_terms);
  float* qpart = (float*)(ws + o_q);
  float* P = (float*)(ws + o_p);
  const int npad = (int)pl.npad;
  L(K_COMPACT, k_compact, dim3(1), dim3(1024), targets, p->target_bytes, pl.n, pl.v, p->ignore_index,
    idx, (int*)(ws + pl.o_pos), nv, n_valid, dev_status, lse_s, lse_t, none ? loss : (float*)nullptr);
  uint16_t* hvt = kd_hvt_bytes(pl, kd.dt) > 0 ? (uint16_t*)(ws + o_hvt) : nullptr;
  if (hvt) launch_gather(L, kd.ht, kd.ldht, kd.dt, npad, idx, nv, hvt);
  for (int64_t s = 0; s < pl.nslab; ++s) {
    const int64_t v0 = s * pl.vc;
    const int vs = (int)(pl.v - v0 < pl.vc ? pl.v - v0 : pl.vc);
    launch_teacher<Z_WRITE>(L, K_KD_Z, kd, hvt, pl, v0, vs, idx, nv, P);
    const int tm = (vs + TILE - 1) / TILE;
    const TileOrder to = tile_order(tm, pl.nt_max, student_group(tm, pl.d));
    L(K_KD_STATS, k_kd_tile<KD_STATS, 2>, dim3(to.grid), dim3(NTHREADS), wsm, pl.ldw, v0, vs, hs, pl.ldh,
      pl.n, (const int*)idx, (const int*)nv, (const float*)nullptr,
      (const float*)nullptr, (const int*)nullptr, p->reduction, (int)pl.d, tm, (uint16_t*)nullptr, (int)pl.vc,
      npad, k.scale2, k.inv_t, P, qpart, to.gw);
    L(K_KD_COMBINE, k_kd_combine, dim3((unsigned)((pl.n + kKdTok - 1) / kKdTok)), dim3(1024), (const float*)qpart,
      tm, (int64_t)npad, qpart + (int64_t)(pl.vc / TILE) * kKdVals * npad, (int)(s == 0), (int)(s + 1 == pl.nslab),
      (const int*)idx, (const int*)nv, lse_s, lse_t, terms, none ? loss : (float*)nullptr);
  }
  if (!none) L(K_LOSS, k_loss, dim3(1), dim3(1024), (const float*)terms, (const int*)nv, p->reduction, loss);
  return L.st;
}

// Forward and backward of the KD loss in one call (the upstream gradient is read on the device
// when the gradient kernels run): the two calls' kernels, with the valid-row list and the teacher's
// gathered rows formed once.
lce_status_t kd_fused_impl(const lce_kd_problem_t* p, const void* Hs, const void* Ws, const void* Ht,
                           const void* Wt, const void* targets, const float* grad_loss, float* loss, float* lse_s,
                           float* lse_t, int32_t* n_valid, int32_t* dev_status, void* dHs, void* dWs,
                           void* workspace, size_t workspace_bytes, void* stream) {
  KdPlan k;
  lce_status_t st = make_kd_plan(p, &k);
  if (st == LCE_OK && workspace_bytes < k.bwd_bytes) st = make_kd_plan(p, &k, true);   // (as backward_impl will)
  if (st != LCE_OK) return st;
  const Plan& pl = k.s;
  if (!loss || !n_valid || !grad_loss || !dWs) return LCE_ERR_NULL;
  if (!aligned16(dWs)) return LCE_ERR_ALIGN;
  if (pl.n > 0 && (!Hs || !Ws || !Ht || !Wt || !targets || !lse_s || !lse_t || !dHs || !workspace))
    return LCE_ERR_NULL;
  if (pl.n > 0 && (!aligned16(Hs) || !aligned16(Ws) || !aligned16(Ht) || !aligned16(Wt) || !aligned16(dHs) ||
                   ((uintptr_t)workspace & 255) != 0))
    return LCE_ERR_ALIGN;
  if (pl.n > 0 && workspace_bytes < k.bwd_bytes) return LCE_ERR_WORKSPACE;
  const bool none = p->reduction == LCE_REDUCE_NONE;
  if (pl.n == 0) {
    Launcher L{(hipStream_t)stream};
    L(K_MISC, k_fwd_empty, dim3(1), dim3(64), none ? (float*)nullptr : loss, n_valid, dev_status);
    if (L.st != LCE_OK) return L.st;
    return backward_impl(&k.ps, nullptr, Hs, Ws, targets, lse_s, n_valid, grad_loss, dHs, nullptr,
                         (uint16_t*)dWs, nullptr, nullptr, workspace, workspace_bytes, stream);
  }
  Launcher L{(hipStream_t)stream};
  const KdArgs kd{(const uint16_t*)Ht, k.t.ldh, (const uint16_t*)Wt, k.t.ldw, (int)k.t.d, lse_t, k.scale2, k.inv_t, true};
  st = kd_forward_launches(L, p, k, kd, (const uint16_t*)Hs, (const uint16_t*)Ws, targets, loss, lse_s, lse_t, n_valid,
                           dev_status, (char*)workspace, pl.o_g, pl.o_dh32, pl.bwd_bytes, pl.bwd_bytes + kd_p_bytes(pl));
  if (st != LCE_OK) return st;
  return backward_impl(&k.ps, nullptr, Hs, Ws, targets, lse_s, n_valid, grad_loss, dHs, nullptr, (uint16_t*)dWs,
                       nullptr, nullptr, workspace, workspace_bytes, stream, &kd);
}

lce_status_t kd_forward_impl(const lce_kd_problem_t* p, const void* Hs, const void* Ws, const void* Ht,
                             const void* Wt, const void* targets, float* loss, float* lse_s, float* lse_t,
                             int32_t* n_valid, int32_t* dev_status, void* workspace, size_t workspace_bytes,
                             void* stream) {
  KdPlan k;
  lce_status_t st = make_kd_plan(p, &k);
  if (st == LCE_OK && workspace_bytes < k.fwd_bytes) st = make_kd_plan(p, &k, true);
  if (st != LCE_OK) return st;
  const Plan& pl = k.s;
  if (!loss || !n_valid) return LCE_ERR_NULL;
  if (pl.n > 0 && (!Hs || !Ws || !Ht || !Wt || !targets || !lse_s || !lse_t || !workspace)) return LCE_ERR_NULL;
  if (pl.n > 0 && (!aligned16(Hs) || !aligned16(Ws) || !aligned16(Ht) || !aligned16(Wt) ||
                   ((uintptr_t)workspace & 255) != 0))
    return LCE_ERR_ALIGN;
  if (pl.n > 0 && workspace_bytes < k.fwd_bytes) return LCE_ERR_WORKSPACE;
  Launcher L{(hipStream_t)stream};
  const bool none = p->reduction == LCE_REDUCE_NONE;
  if (pl.n == 0) {
    L(K_MISC, k_fwd_empty, dim3(1), dim3(64), none ? (float*)nullptr : loss, n_valid, dev_status);
    return L.st;
  }
  const KdArgs kd{(const uint16_t*)Ht, k.t.ldh, (const uint16_t*)Wt, k.t.ldw, (int)k.t.d, nullptr, k.scale2, k.inv_t, false};
  return kd_forward_launches(L, p, k, kd, (const uint16_t*)Hs, (const uint16_t*)Ws, targets, loss, lse_s, lse_t, n_valid,
                             dev_status, (char*)workspace, k.o_q, k.o_terms, k.o_p, k.o_hvt);
}

}  // namespace

extern "C" {

const char* lce_status_string(lce_status_t s) {
  switch (s) {
    case LCE_OK: return "ok";
    case LCE_ERR_NULL: return "required pointer is NULL";
    case LCE_ERR_SHAPE: return "invalid or too large shape / stride";
    case LCE_ERR_ALIGN: return "pointer, stride or workspace misaligned";
    case LCE_ERR_UNSUPPORTED: return "unsupported configuration (d % 8, reduction or target width)";
    case LCE_ERR_WORKSPACE: return "workspace too small";
    case LCE_ERR_HIP: return "HIP runtime or kernel launch failure";
    case LCE_ERR_ARG: return "invalid argument";
  }
  return "unknown status";
}

lce_status_t lce_plan_info(const lce_problem_t* p, lce_plan_info_t* out) {
  Plan pl;
  lce_status_t st = make_plan(p, &pl);
  if (st != LCE_OK) return st;
  if (!out) return LCE_ERR_NULL;
  out->npad = pl.npad;
  out->rows_g = pl.rows_g;
  out->vc = pl.vc;
  out->nslab = pl.nslab;
  out->dh_kz = pl.dh_kz;
  out->part_rows = pl.part_rows;
  out->fwd_gathers = 1;
  out->fwd_one_launch = pl.one_launch ? 1 : 0;
  out->o_idx = (int64_t)pl.o_idx;
  out->o_pos = (int64_t)pl.o_pos;
  out->o_nv = (int64_t)pl.o_nv;
  out->o_hv = (int64_t)pl.o_hv;
  out->o_pm = (int64_t)pl.o_pm;
  out->o_ps = (int64_t)pl.o_ps;
  out->o_terms = (int64_t)pl.o_terms;
  out->fwd_bytes = (int64_t)pl.fwd_bytes;
  out->o_g = (int64_t)pl.o_g;
  out->o_dh32 = (int64_t)pl.o_dh32;
  out->o_dh32b = (int64_t)pl.o_dh32b;
  out->bwd_bytes = (int64_t)pl.bwd_bytes;
  return LCE_OK;
}

// The device address of `scratch` on the current device, taken once per device (with that
// device current) and kept: every call on a GPU then shares that GPU's copy.
struct ScratchAddrs {
  std::mutex mu;
  static constexpr int kMaxDevices = 64;
  void* ptr[kMaxDevices] = {};
};
ScratchAddrs g_scratch;

lce_status_t noalloc_scratch(void* stream, void** out) {
  int dev = -1;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= ScratchAddrs::kMaxDevices) return LCE_ERR_HIP;
  if (stream) {
    hipDevice_t sdev = -1;
    if (hipStreamGetDevice((hipStream_t)stream, &sdev) != hipSuccess) return LCE_ERR_HIP;
    if (sdev != dev) return LCE_ERR_ARG;   // the stream must belong to the current device
  }
  std::lock_guard<std::mutex> lk(g_scratch.mu);
  if (!g_scratch.ptr[dev]) {
    void* a = nullptr;
    if (hipGetSymbolAddress(&a, HIP_SYMBOL(scratch)) != hipSuccess || !a) return LCE_ERR_HIP;
    g_scratch.ptr[dev] = a;
  }
  *out = g_scratch.ptr[dev];
  return LCE_OK;
}

lce_status_t lce_workspace_size(const lce_problem_t* p, size_t* fwd_bytes, size_t* bwd_bytes) {
  Plan pl;
  lce_status_t st = make_plan(p, &pl);
  if (st != LCE_OK) return st;
  if (fwd_bytes) *fwd_bytes = pl.fwd_bytes;
  if (bwd_bytes) *bwd_bytes = pl.bwd_bytes;
  return LCE_OK;
}

lce_status_t lce_workspace_size_least(const lce_problem_t* p, size_t* fwd_bytes, size_t* bwd_bytes) {
  Plan pl;
  lce_status_t st = make_plan(p, &pl);
  if (st != LCE_OK) return st;
  if (fwd_bytes) {
    const size_t full = pl.fwd_bytes;
    plan_forward(&pl, true);
    *fwd_bytes = std::min(full, pl.fwd_bytes);
  }
  if (bwd_bytes) {
    plan_backward(&pl, true);
    *bwd_bytes = pl.bwd_bytes;
  }
  return LCE_OK;
}

lce_status_t lce_forward(const lce_problem_t* p, const void* H, const void* W, const void* targets,
                         float* loss, float* lse, int32_t* n_valid, int32_t* dev_status,
                         void* workspace, size_t workspace_bytes, void* stream) {
  return forward_impl(p, nullptr, H, W, targets, loss, lse, nullptr, n_valid, dev_status, workspace,
                      workspace_bytes, stream);
}

lce_status_t lce_forward_noalloc(const lce_problem_t* p, const void* H, const void* W, const void* targets,
                                 float* loss, float* lse, int32_t* n_valid, int32_t* dev_status, void* stream) {
  Plan pl;
  lce_status_t st = make_plan(p, &pl);
  if (st != LCE_OK) return st;
  if (pl.fwd_bytes > (size_t)LCE_NOALLOC_SCRATCH_BYTES) return LCE_ERR_WORKSPACE;
  void* ws = nullptr;
  st = noalloc_scratch(stream, &ws);
  if (st != LCE_OK) return st;
  // nothing of the previous call's contents is read: every region is written before it is used
  return forward_impl(p, nullptr, H, W, targets, loss, lse, nullptr, n_valid, dev_status, ws,
                      (size_t)LCE_NOALLOC_SCRATCH_BYTES, stream);
}

lce_status_t lce_forward_shard(const lce_problem_t* p, const lce_shard_t* shard, const void* H, const void* W,
                               const void* targets, float* lse_part, float* tgt_part, int32_t* n_valid,
                               int32_t* dev_status, void* workspace, size_t workspace_bytes, void* stream) {
  ShardInfo si;
  lce_status_t st = shard_info(p, shard, &si);
  if (st != LCE_OK) return st;
  return forward_impl(p, &si, H, W, targets, nullptr, lse_part, tgt_part, n_valid, dev_status, workspace,
                      workspace_bytes, stream);
}

lce_status_t lce_combine_shards(const lce_problem_t* p, int32_t n_shards, const float* lse_parts,
                                const float* tgt_parts, const void* targets, float* loss, float* lse,
                                int32_t* n_valid, int32_t* dev_status, void* workspace, size_t workspace_bytes,
                                void* stream) {
  Plan pl;
  lce_status_t st = make_plan(p, &pl);
  if (st != LCE_OK) return st;
  if (n_shards < 1 || n_shards > 4096) return LCE_ERR_ARG;
  if (!loss || !n_valid) return LCE_ERR_NULL;
  if (pl.n > 0 && (!lse_parts || !tgt_parts || !targets || !lse || !workspace)) return LCE_ERR_NULL;
  if (pl.n > 0 && ((uintptr_t)workspace & 255) != 0) return LCE_ERR_ALIGN;
  if (pl.n > 0 && !forward_fits(&pl, workspace_bytes)) return LCE_ERR_WORKSPACE;
  Launcher L{(hipStream_t)stream};
  const bool none = p->reduction == LCE_REDUCE_NONE;
  if (pl.n == 0) {
    L(K_MISC, k_fwd_empty, dim3(1), dim3(64), none ? (float*)nullptr : loss, n_valid, dev_status);
    return L.st;
  }
  char* ws = (char*)workspace;
  int* idx = (int*)(ws + pl.o_idx);
  int* pos = (int*)(ws + pl.o_pos);
  int* nv = (int*)(ws + pl.o_nv);
  float* terms = (float*)(ws + pl.o_terms);
  L(K_COMPACT, k_compact, dim3(1), dim3(1024), targets, p->target_bytes, pl.n, pl.v, p->ignore_index,
    idx, pos, nv, n_valid, dev_status, lse, none ? loss : (float*)nullptr, (float*)nullptr);
  L(K_SHARD_COMBINE, k_shard_combine, dim3((unsigned)((pl.n + 255) / 256)), dim3(256), (int)n_shards, lse_parts,
    tgt_parts, pl.n, (const int*)idx, (const int*)nv, lse, terms, none ? loss : (float*)nullptr);
  if (!none) L(K_LOSS, k_loss, dim3(1), dim3(1024), (const float*)terms, (const int*)nv, p->reduction, loss);
  return L.st;
}

lce_status_t lce_backward(const lce_problem_t* p, const void* H, const void* W, const void* targets,
                          const float* lse, const int32_t* n_valid, const float* grad_loss,
                          void* dH, void* dW, void* workspace, size_t workspace_bytes, void* stream) {
  if (!dW) return LCE_ERR_NULL;
  if (!aligned16(dW)) return LCE_ERR_ALIGN;
  return backward_impl(p, nullptr, H, W, targets, lse, n_valid, grad_loss, dH, nullptr, (uint16_t*)dW, nullptr,
                       nullptr, workspace, workspace_bytes, stream);
}

lce_status_t lce_backward_select(const lce_problem_t* p, const void* H, const void* W, const void* targets,
                                 const float* lse, const int32_t* n_valid, const float* grad_loss,
                                 void* dH, void* dW, void* workspace, size_t workspace_bytes, void* stream) {
  if (!dH && !dW) return LCE_ERR_NULL;
  if (!aligned16(dH) || !aligned16(dW)) return LCE_ERR_ALIGN;
  return backward_impl(p, nullptr, H, W, targets, lse, n_valid, grad_loss, dH, nullptr, (uint16_t*)dW, nullptr,
                       nullptr, workspace, workspace_bytes, stream, nullptr,
                       (dH ? WANT_DH : 0) | (dW ? WANT_DW : 0));
}

lce_status_t lce_backward_shard(const lce_problem_t* p, const lce_shard_t* shard, const void* H, const void* W,
                                const void* targets, const float* lse, const int32_t* n_valid,
                                const float* grad_loss, float* dH_part, void* dW, void* workspace,
                                size_t workspace_bytes, void* stream) {
  ShardInfo si;
  lce_status_t st = shard_info(p, shard, &si);
  if (st != LCE_OK) return st;
  if (!dW || (p->n > 0 && !dH_part)) return LCE_ERR_NULL;
  if (!aligned16(dW)) return LCE_ERR_ALIGN;
  return backward_impl(p, &si, H, W, targets, lse, n_valid, grad_loss, nullptr, dH_part, (uint16_t*)dW, nullptr,
                       nullptr, workspace, workspace_bytes, stream);
}

lce_status_t lce_adamw_step(int64_t v, int64_t d, int64_t ld_w, void* W, const void* dW, float* exp_avg,
                            float* exp_avg_sq, float* W_master, const lce_adamw_t* opt, void* stream) {
  AdamWConst c;
  lce_status_t st = make_adamw(opt, &c);
  if (st != LCE_OK) return st;
  const int64_t ldw = ld_w ? ld_w : d;
  if (v < 1 || d < 8 || ldw < d || v >= (int64_t)1 << 30 || d >= (int64_t)1 << 20) return LCE_ERR_SHAPE;
  if (d % 8 != 0) return LCE_ERR_UNSUPPORTED;
  if (ldw % 8 != 0) return LCE_ERR_ALIGN;
  if (!W || !exp_avg || !exp_avg_sq) return LCE_ERR_NULL;
  if (!aligned16(W) || !aligned16(exp_avg) || !aligned16(exp_avg_sq) || (dW && !aligned16(dW)) ||
      (W_master && !aligned16(W_master)))
    return LCE_ERR_ALIGN;
  AdamWState as{(uint16_t*)W, ldw, exp_avg, exp_avg_sq, W_master};
  Launcher L{(hipStream_t)stream};
  L(K_ADAMW, k_adamw, dim3(adamw_grid(v, d)), dim3(256), v, (int)d, (const uint16_t*)dW, as, c);
  return L.st;
}

lce_status_t lce_backward_adamw(const lce_problem_t* p, const void* H, void* W, const void* targets,
                                const float* lse, const int32_t* n_valid, const float* grad_loss, void* dH,
                                float* exp_avg, float* exp_avg_sq, float* W_master, const lce_adamw_t* opt,
                                void* workspace, size_t workspace_bytes, void* stream) {
  AdamWConst c;
  lce_status_t st = make_adamw(opt, &c);
  if (st != LCE_OK) return st;
  if (!p) return LCE_ERR_NULL;
  if (p->flags & LCE_FLAG_ACCUMULATE_DW) return LCE_ERR_ARG;
  if (!exp_avg || !exp_avg_sq) return LCE_ERR_NULL;
  if (!aligned16(exp_avg) || !aligned16(exp_avg_sq) || (W_master && !aligned16(W_master))) return LCE_ERR_ALIGN;
  AdamWState as{(uint16_t*)W, p->ld_w ? p->ld_w : p->d, exp_avg, exp_avg_sq, W_master};
  return backward_impl(p, nullptr, H, W, targets, lse, n_valid, grad_loss, dH, nullptr, nullptr, &as, &c,
                       workspace, workspace_bytes, stream);
}

lce_status_t lce_kd_workspace_size(const lce_kd_problem_t* p, size_t* fwd_bytes, size_t* bwd_bytes) {
  KdPlan k;
  lce_status_t st = make_kd_plan(p, &k);
  if (st != LCE_OK) return st;
  if (fwd_bytes) *fwd_bytes = k.fwd_bytes;
  if (bwd_bytes) *bwd_bytes = k.bwd_bytes;
  return LCE_OK;
}

lce_status_t lce_kd_workspace_size_least(const lce_kd_problem_t* p, size_t* fwd_bytes, size_t* bwd_bytes) {
  KdPlan k;
  lce_status_t st = make_kd_plan(p, &k, true);
  if (st != LCE_OK) return st;
  if (fwd_bytes) *fwd_bytes = k.fwd_bytes;
  if (bwd_bytes) *bwd_bytes = k.bwd_bytes;
  return LCE_OK;
}

lce_status_t lce_kd_forward(const lce_kd_problem_t* p, const void* Hs, const void* Ws, const void* Ht,
                            const void* Wt, const void* targets, float* loss, float* lse_s, float* lse_t,
                            int32_t* n_valid, int32_t* dev_status, void* workspace, size_t workspace_bytes,
                            void* stream) {
  return kd_forward_impl(p, Hs, Ws, Ht, Wt, targets, loss, lse_s, lse_t, n_valid, dev_status, workspace,
                         workspace_bytes, stream);
}

lce_status_t lce_kd_forward_backward(const lce_kd_problem_t* p, const void* Hs, const void* Ws, const void* Ht,
                                     const void* Wt, const void* targets, const float* grad_loss, float* loss,
                                     float* lse_s, float* lse_t, int32_t* n_valid, int32_t* dev_status, void* dHs,
                                     void* dWs, void* workspace, size_t workspace_bytes, void* stream) {
  return kd_fused_impl(p, Hs, Ws, Ht, Wt, targets, grad_loss, loss, lse_s, lse_t, n_valid, dev_status, dHs, dWs,
                       workspace, workspace_bytes, stream);
}

lce_status_t lce_kd_workspace_size_fused(const lce_kd_problem_t* p, size_t* bytes) {
  KdPlan k;
  lce_status_t st = make_kd_plan(p, &k);
  if (st != LCE_OK) return st;
  if (bytes) *bytes = k.bwd_bytes;
  return LCE_OK;
}

lce_status_t lce_kd_backward(const lce_kd_problem_t* p, const void* Hs, const void* Ws, const void* Ht,
                             const void* Wt, const void* targets, const float* lse_s, const float* lse_t,
                             const int32_t* n_valid, const float* grad_loss, void* dHs, void* dWs,
                             void* workspace, size_t workspace_bytes, void* stream) {
  KdPlan k;
  lce_status_t st = make_kd_plan(p, &k);
  if (st != LCE_OK) return st;
  if (!dWs) return LCE_ERR_NULL;
  if (!aligned16(dWs)) return LCE_ERR_ALIGN;
  if (p->n > 0 && (!Ht || !Wt || !lse_t)) return LCE_ERR_NULL;
  if (p->n > 0 && (!aligned16(Ht) || !aligned16(Wt))) return LCE_ERR_ALIGN;
  const KdArgs kd{(const uint16_t*)Ht, k.t.ldh, (const uint16_t*)Wt, k.t.ldw, (int)k.t.d, lse_t, k.scale2, k.inv_t,
                  false};
  return backward_impl(&k.ps, nullptr, Hs, Ws, targets, lse_s, n_valid, grad_loss, dHs, nullptr, (uint16_t*)dWs,
                       nullptr, nullptr, workspace, workspace_bytes, stream, &kd);
}

lce_status_t lce_timing_enable(int on) {
  std::lock_guard<std::mutex> lk(g_timing.mu);
  if (on) {
    if (g_timing.ev.empty()) {
      g_timing.ev.resize(2 * Timing::kPool);
      g_timing.kind.assign(Timing::kPool, 0);
      for (auto& e : g_timing.ev)
        if (hipEventCreate(&e) != hipSuccess) {
          g_timing.ev.clear();
          return LCE_ERR_HIP;
        }
    }
    g_timing.used = 0;
    g_timing.on = true;
  } else {
    g_timing.on = false;
  }
  return LCE_OK;
}

int lce_timing_kernel_count(void) { return K_COUNT; }

const char* lce_timing_kernel_name(int k) { return (k >= 0 && k < K_COUNT) ? kKernelNames[k] : nullptr; }

lce_status_t lce_timing_read(int k, double* total_ms, int64_t* launches) {
  if (k < 0 || k >= K_COUNT) return LCE_ERR_ARG;
  if (!total_ms || !launches) return LCE_ERR_NULL;
  std::lock_guard<std::mutex> lk(g_timing.mu);
  double tot = 0.0;
  int64_t cnt = 0;
  for (int i = 0; i < g_timing.used; ++i) {
    if (g_timing.kind[i] != k) continue;
    if (hipEventSynchronize(g_timing.ev[2 * i + 1]) != hipSuccess) return LCE_ERR_HIP;
    float ms = 0.f;
    if (hipEventElapsedTime(&ms, g_timing.ev[2 * i], g_timing.ev[2 * i + 1]) != hipSuccess) return LCE_ERR_HIP;
    tot += ms;
    ++cnt;
  }
  *total_ms = tot;
  *launches = cnt;
  return LCE_OK;
}

}  // extern "C"
