// bf16 MFMA grouped GEMMs of the SwiGLU expert FFN, forward and backward
// (Sec. 3.2.5 SwiGLU among the efficient kernels; App. B.6 stacked expert-major weights).
//
// One kernel skeleton serves all nine matrix products of the layer (and the three of the router):
//   * a BM x BN output tile per workgroup, a grid of WGM x WGN wavefronts over it, each owning a
//     WM x WN sub-tile made of 16x16 MFMA tiles (v_mfma_f32_16x16x32_bf16, fp32 accumulators kept in
//     registers for the whole reduction); the default is 256 x 256 with 2 x 4 wavefronts of 128 x 64;
//   * the reduction dimension is walked in BK-wide slabs through two LDS rings (one per operand) that are
//     filled by direct global->LDS loads (no staging registers); one to two slabs are in flight behind the
//     one being multiplied, every MFMA operand is read from LDS most of a reduction step before its use,
//     and one barrier per slab separates writers from readers; what does not exist (rows, columns, the end
//     of a partial last slab) is out of the loads' range and reads as zero;
//   * a workgroup stays on its CU and takes tile after tile: the first two slabs of the next tile are enqueued
//     behind the last of this one and land while the epilogue runs;
//   * results leave through LDS as well -- 16 rows of a wave at a time, in the one ring buffer that is free
//     between two tiles -- so that all global stores (and the loads of the saved pre-activations in the fused
//     SwiGLU derivative) are 16 bytes per lane and contiguous along rows;
//   * an operand whose reduction index is contiguous in memory is staged as
//     [rows][BK] and read with 16-byte LDS loads; an operand whose reduction index is the
//     slow axis in memory (the weight in the two backward-data products, both operands of
//     the weight-gradient products) is staged untransposed as [BK][rows] and read with
//     the transposing LDS load ds_read_b64_tr_b16, which hands every lane four
//     consecutive reduction elements of its own row.  Both layouts are XOR-swizzled so
//     that each group of lanes the LDS serves in one cycle covers all 64 banks.
// Row-grouped products (rows of the activation matrix belong to experts) take their
// (expert, row-tile) list from a small schedule built on the device from `offsets`, so no
// host synchronisation is needed.  Weight-gradient products reduce over an expert's rows
// instead: a second device-built schedule cuts long experts into bounded chunks whose fp32
// partial tiles a small kernel adds in chunk order (no float atomics).
// Workgroup ids are remapped so that consecutive tiles -- which share an expert's weights
// -- run on the same XCD (workgroup b runs on XCD b mod 8) and hit its L2.
// The router linear (logits, its weight gradient, its part of the input gradient) runs on
// the same skeleton with a single segment of all rows.
#include <algorithm>
#include <mutex>
#include <type_traits>
#include <utility>
#include "launch_plan.h"
#include "moe_common.h"

namespace moe {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));

// ---- tile shapes ------------------------------------------------------------------------------
template <int BM_, int BN_, int BK_, int WGM_, int WGN_, int STAGES_A_, int STAGES_B_>
struct Tile {
  static constexpr int BM = BM_, BN = BN_, BK = BK_;
  static constexpr int WGM = WGM_, WGN = WGN_;            // grid of wavefronts over the tile
  static constexpr int kWaves = WGM * WGN, kThreads = 64 * kWaves;
  static constexpr int WM = BM / WGM, WN = BN / WGN;      // sub-tile of one wavefront
  static constexpr int MI = WM / 32, NI = WN / 32;        // 32-row strips and 32-column stretches per wave
  static constexpr int FM = WM / 16, FN = WN / 16;        // bf16 MFMA fragments per wave (16 x 16 outputs each)
  static constexpr int kABytes = BM * BK * 2, kBBytes = BN * BK * 2;
  // LDS ring: each operand has its own ring of slab buffers (SA for the row side, SB for the column side); slab kt
  // lives in buffer kt % SA and kt % SB.  One slab is being multiplied, the others are in flight.  With 64 KiB per
  // slab only 2.5 slabs fit the 160 KiB of a CU: SA = 2, SB = 3, which is what keeps the CU's window of outstanding
  // L2 requests full across the barrier that separates two slabs (with 2 + 2 it drains at every slab).  The deeper
  // ring goes to the side with fewer fragments per wave: its third buffer lies beyond the 16-bit immediate offset of
  // the LDS instructions and costs one more address register per fragment.
  static constexpr int SA = STAGES_A_, SB = STAGES_B_;
  static constexpr int kBBase = SA * kABytes;             // the column side's buffers follow the row side's
  static constexpr int kLdsBytes = SA * kABytes + SB * kBBytes;
  static_assert(kLdsBytes <= 160 * 1024, "a CU has 160 KiB of LDS");
  static constexpr int kBlocksPerCu = 2 * kLdsBytes <= 160 * 1024 ? 2 : 1;   // by LDS capacity
  static constexpr int kWavesPerSimd = kBlocksPerCu * kWaves / 4;
};

// Hands back its argument through an empty asm: values derived from the result cannot be computed before
// this point, so per-lane indices of the epilogue and of the next tile's loads do not occupy registers during the main loop.
__device__ __forceinline__ int not_before_here(int v) { asm volatile("" : "+v"(v)); return v; }
// A wave-uniform value in a scalar register (integer divisions and clamps are done on the vector unit, and everything derived
// from their results would stay there).
__device__ __forceinline__ int scalar(int v) { return __builtin_amdgcn_readfirstlane(not_before_here(v)); }
// This lane of the wave, worked out where it is wanted: threadIdx.x kept for it would occupy a register during the main loop.
__device__ __forceinline__ int lane_id() {
  unsigned all = ~0u;
  asm volatile("" : "+s"(all));
  return static_cast<int>(__builtin_amdgcn_mbcnt_hi(all, __builtin_amdgcn_mbcnt_lo(all, 0u)));
}
// min of two wave-uniform values, as a scalar instruction (a minimum and a maximum in a row would become one vector instruction)
__device__ __forceinline__ int scalar_min(int a, int b) {
  int v = min(a, b);
  asm("" : "+s"(v));
  return v;
}

// One operand tile of ROWS rows: element (row, k).  Two halves of ROWS/2 rows with their own
// base so that the gate and the up projection can share one tile.
//   k-contiguous: half[h] + row * ld + k          k-strided: half[h] + k * ld + row
struct Operand {
  const bf16_t* half[2];
  long ld;
  int valid[2];      // rows of each half that exist (others read as zero); multiples of 8 if k-strided
  // Gathered operands (the matrix is [*, ld] and never copied into expert order): logical row r of the
  // operand -- a tile row if k-contiguous, a reduction index if k-strided -- is memory row gather[grow + r]
  // of half[0]; half[1] is not used, and every byte offset (row * ld * 2) must fit in 32 bits.
  const int32_t* gather;
  int grow;
};

// ---- LDS layouts ---------------------------------------------------------------------------------
// k-contiguous operand: [ROWS][BK]; the 16-byte pieces of a row are XORed with the index of the
// 256-byte line the row lives in, so 16 consecutive rows read at one piece index hit 64 banks.
template <int BK>
__device__ __forceinline__ int kc_off(int row, int piece) {
  constexpr int PPR = BK / 8;                    // pieces per row
  constexpr int RPL = 256 / (BK * 2);            // rows per 256-byte line
  return row * (BK * 2) + ((piece ^ ((row / RPL) & (PPR - 1))) << 4);
}
// k-strided operand: [BK][ROWS]; the 32-byte chunks of a k-row (16 columns, what one group of 16 lanes of a transposing
// read takes from it) are XORed with bits 0, 1 and 3 of k, so the eight k-rows that 32 lanes touch together -- four
// consecutive ones from k = 8 g and four from 8 (g + 1) -- lie in different banks.
__device__ __forceinline__ int ks_swizzle(int k) { return ((k & 3) << 1) | ((k >> 3) & 1); }
template <int ROWS>
__device__ __forceinline__ int ks_off(int k, int piece) {
  static_assert(ROWS >= 128, "the swizzle moves a piece by up to 14 pieces of its k-row");
  return k * (ROWS * 2) + ((piece ^ (ks_swizzle(k) << 1)) << 4);
}

// ---- MFMA operand fragments ----------------------------------------------------------------------------
// bf16 fragment = 16 rows x 32 k: lane l holds row l%16, k = 8*(l/16) .. +7 of the 32-wide step kk.
// frag_off: this lane's byte offset inside the operand tile, computed once per kernel; the main loop derives the
// other steps and fragments with compile-time offsets.
template <bool KS, int ROWS, int BK>
__device__ __forceinline__ int frag_off(int row_base, int kk, int lane) {
  if constexpr (!KS) {
    return kc_off<BK>(row_base + (lane & 15), 4 * kk + (lane >> 4));
  } else {
    // Transposing read: within each group of 16 lanes, lane i receives element i%4 of the 8-byte
    // rows addressed by lanes i/4, i/4+4, i/4+8, i/4+12.  Lane s therefore addresses k-row s/4 at
    // columns 4*(s%4)..+3 of the fragment's 16 columns, and ends up with 4 consecutive k of column s.
    const int s = lane & 15;
    const int col = row_base + 4 * (s & 3);                               // multiple of 4
    const int k = kk * 32 + 8 * (lane >> 4) + (s >> 2);
    return ks_off<ROWS>(k, col >> 3) + (col & 4) * 2;                     // 8-byte half of the piece
  }
}
// the fragment of the 8-bit products: 32 rows, lane l holds row l%32, 16-byte piece 2*kk + l/32 (k-contiguous tiles only)
template <int BK>
__device__ __forceinline__ int frag_off_32(int row_base, int kk, int lane) {
  return kc_off<BK>(row_base + (lane & 31), 2 * kk + (lane >> 5));
}
// One fragment: 16 bytes per lane at LDS address `addr` + IMM (a compile-time constant: buffer, reduction step or
// fragment).  Both kinds of read are assembly statements on purpose.
//   * The compiler orders every LDS read it knows to be one behind all outstanding direct global->LDS loads (it
//     cannot tell which bytes they will write): it puts a wait for *all* of this wave's loads in front of the first
//     such read of every slab, which serialises the ring -- the slabs just requested would have to land before the
//     slab in hand may be read.  The ring needs no such wait: a buffer is read only after the counted wait and the
//     barrier that follow its own loads.
//   * The address register and the 16-bit immediate are chosen here, so no address arithmetic is left in the slab
//     loop (every vector instruction there takes issue slots from the MFMAs of both waves of the SIMD).
// The results arrive asynchronously; they are consumed only after a wait that names them as operands (arrived,
// arrived_with_b, all_arrived in MainLoop).
template <bool KS, int ROWS, int IMM>
__device__ __forceinline__ bf16x8 lds_read_frag(uint32_t addr) {
  static_assert(IMM >= 0 && IMM + (KS ? 4 * ROWS * 2 : 0) < 65536, "the immediate offset of an LDS instruction has 16 bits");
  if constexpr (!KS) {
    bf16x8 v;
    asm volatile("ds_read_b128 %0, %1 offset:%2" : "=v"(v) : "v"(addr), "n"(IMM));
    return v;
  } else {
    // k + 4 has the same swizzle (bits 0, 1 and 3 of k unchanged): a constant 4 k-rows further
    bf16x4 lo, hi;
    asm volatile("ds_read_b64_tr_b16 %0, %1 offset:%2" : "=v"(lo) : "v"(addr), "n"(IMM));
    asm volatile("ds_read_b64_tr_b16 %0, %1 offset:%2" : "=v"(hi) : "v"(addr), "n"(IMM + 4 * ROWS * 2));
    return __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
  }
}

// ---- global -> LDS without passing through registers -----------------------------------------------
// One wave instruction (buffer_load_dwordx4 ... lds) moves 64 x 16 bytes into 1 KiB of consecutive LDS;
// the swizzles above are applied on the global side: each lane fetches the piece that belongs in its
// LDS slot.  Addresses are a wave-uniform base in a buffer descriptor (moved on per slab with scalar arithmetic) plus a
// 32-bit per-lane offset.  The descriptor's range check replaces branches and selects: a load beyond it touches no
// memory and writes zeros, so
//   * rows (k-contiguous) or columns (k-strided) that do not exist carry an offset beyond every range,
//   * reduction rows beyond K of a k-strided operand lie beyond the range of the last slab's descriptor, and
//   * slabs beyond the end of the reduction get an empty descriptor,
// and every wave enqueues the same number of loads per slab whatever is left: all waits are immediates and the slab
// loop has a single path.  Only a partial last slab of a k-contiguous operand needs a select (mask_beyond).
//
// Ranges.  k-contiguous: everything but the offset that stands for "does not exist" (token rows of a gathered operand
// reach up to 4 GiB - 128 bytes: the 8-bit products' codes).  Gathered k-strided: a row that does not exist is moved to the
// range's end and a column's offset (below 64 KiB) comes on top, so the range leaves that much room below 4 GiB; its
// operands, the bf16 token matrices, are smaller than that.
// Everything per lane is selected, never branched over: around a divergent branch the compiler rewrites the tile loop's own
// (uniform) branches as lane masks, the parts of the descriptors end up in vector registers, and every load of the slab loop
// becomes a loop over lanes.
__device__ __forceinline__ uint32_t off_if(bool exists, uint32_t off, uint32_t none) {
  asm("" : "+v"(off));                                 // (formed on every path)
  return exists ? off : none;
}
constexpr uint32_t kRangeAll = 0xFFFFFF80u;
constexpr uint32_t kRangeRows = 0xFFFF0000u;
constexpr uint32_t kOffNone = 0xFFFFFFF0u;      // beyond every range
template <bool KS, int ROWS, int BK, int WAVES, bool GATHER = false, bool TWO_SEG = false> struct Dma {
  static constexpr int CHUNKS = ROWS * BK * 2 / 1024;
  static constexpr int N = CHUNKS / WAVES;                   // chunks per wave
  static_assert(N >= 1 && CHUNKS % WAVES == 0, "tile too small for this many waves");
  static_assert(WAVES % 2 == 0, "a wave's chunks must lie in one half of the tile");
  static constexpr int KPC = KS ? 1024 / (ROWS * 2) : 1;      // k-strided: reduction rows per chunk
  static constexpr int NR = N * KPC;                         // k-strided: reduction rows per wave and slab (consecutive)
  const char* base;          // wave-uniform: slab 0
  long step;                 // bytes per slab (uniform)
  uint32_t voff[N];          // per lane, bytes
  int K, nslabs;             // reduction length of a segment (k-strided: limits its last slab) and slabs that exist
  int seg_slabs;             // TWO_SEG: slabs seg_slabs.. belong to a second segment ...
  long seg_delta;            // ... whose bytes lie this much further
  int valid;                 // k-contiguous: rows of this wave's half of the tile that exist
  __amdgpu_buffer_rsrc_t rsrc;   // the slab being enqueued
  // The row list of a gathered operand.  k-strided: the memory rows of the wave's NR reduction rows of the next slab to be issued,
  // fetched one slab ahead with scalar loads, which do not touch the vector-memory counter that orders the ring.  k-contiguous: the
  // memory rows of the wave's tile rows, once per tile; every lane wants its own, so these are vector loads, and the wait for
  // them is one for everything in flight (as scalar loads, eight rows at a time: gate/up 394 -> 399 us).
  typedef __attribute__((address_space(4))) const int32_t* RowList;
  typedef int32_t RowVec __attribute__((ext_vector_type(KS && GATHER ? NR : 1)));   // a value, not an array: stays in scalar registers
  RowList rows;              // wave-uniform: gather + grow + wave * NR
  RowVec next_row;
  uint32_t ld2;              // bytes per memory row
  int lq;                    // per lane: which of the KPC rows of a chunk this lane loads
  int k_first;               // k-strided: first reduction row of this wave inside a slab
  __device__ __forceinline__ void fetch_rows(int slab) {
    if constexpr (KS && GATHER) {
      RowList r = rows + slab * BK;
#pragma unroll
      for (int j = 0; j < NR; ++j) next_row[j] = r[j];
    }
  }
  // k-contiguous: this lane's 16-byte piece of chunk i
  static __device__ __forceinline__ void place_of(int i, int wave, int lane, int& row, int& piece) {
    constexpr int PPR = BK / 8, RPC = 1024 / (BK * 2), RPL = 256 / (BK * 2);
    row = (wave * N + i) * RPC + lane / PPR;
    piece = (lane % PPR) ^ ((row / RPL) & (PPR - 1));
  }
  // k-contiguous, in row order: the offsets of every chunk
  __device__ __forceinline__ void place_rows(int wave, int lane) {
    static_assert(!KS && !GATHER, "");
#pragma unroll
    for (int i = 0; i < N; ++i) {
      int row, piece;
      place_of(i, wave, lane, row, piece);
      const int rh = row - (wave >= WAVES / 2 ? ROWS / 2 : 0);
      voff[i] = off_if(rh < valid, static_cast<uint32_t>(rh) * ld2 + piece * 16, kOffNone);
    }
  }
  // point at an operand of another tile.  K_: reduction length (of a segment), nslabs_: slabs that exist
  __device__ __forceinline__ void init(const Operand& op, int K_, int nslabs_, int wave, int lane) {
    K = K_; nslabs = nslabs_;
    asm("" : "+s"(K), "+s"(nslabs));                          // scalar registers on every path: the descriptors are made of them
    ld2 = static_cast<uint32_t>(op.ld * 2);
    const bf16_t* b = op.half[0];
    if constexpr (!KS) {
      const bool upper = wave >= WAVES / 2;                    // uniform
      valid = upper ? op.valid[1] : op.valid[0];
      if constexpr (GATHER) {
        constexpr int PPR = BK / 8, RPC = 1024 / (BK * 2);
        RowList r = reinterpret_cast<RowList>(reinterpret_cast<uintptr_t>(op.gather + op.grow + wave * (N * RPC)));
#pragma unroll
        for (int i = 0; i < N; ++i) {
          int row, piece, mrow = r[i * RPC];
          place_of(i, wave, lane, row, piece);
#pragma unroll
          for (int q = 1; q < RPC; ++q) mrow = lane / PPR == q ? r[i * RPC + q] : mrow;   // entries past the tile's rows exist (padding) and are not used
          voff[i] = off_if(row - (upper ? ROWS / 2 : 0) < valid, static_cast<uint32_t>(mrow) * ld2 + piece * 16, kOffNone);
        }
      } else {
        if (upper) b = op.half[1];
        place_rows(wave, lane);
      }
    } else {
      constexpr int PPK = ROWS / 8;
#pragma unroll
      for (int i = 0; i < N; ++i) {
        const int k = (wave * N + i) * KPC + lane / PPK;
        const int piece = (lane % PPK) ^ (ks_swizzle(k) << 1);
        const int col = piece * 8;
        const bool exists = col < op.valid[0] + op.valid[1];   // k-strided operands are never dual
        // (gathered: a column that does not exist reads the row's first one, so that row offset + column offset cannot wrap)
        if constexpr (GATHER) voff[i] = off_if(exists, col * 2, 0);
        else voff[i] = off_if(exists, static_cast<uint32_t>(k) * ld2 + col * 2, kOffNone);
      }
    }
    step = (KS ? (GATHER ? 0L : static_cast<long>(BK) * op.ld) : BK) * 2;
    // the base is the same in every lane: say so
    const uint64_t b64 = reinterpret_cast<uint64_t>(b);
    const uint32_t lo = __builtin_amdgcn_readfirstlane(static_cast<uint32_t>(b64));
    const uint32_t hi = __builtin_amdgcn_readfirstlane(static_cast<uint32_t>(b64 >> 32));
    base = reinterpret_cast<const char*>((static_cast<uint64_t>(hi) << 32) | lo);
    if constexpr (KS && GATHER) {
      rows = reinterpret_cast<RowList>(reinterpret_cast<uintptr_t>(op.gather + op.grow + wave * NR));
      lq = lane / (ROWS / 8);
      k_first = wave * NR;
      fetch_rows(0);
    }
  }
  // the partial last slab of a segment of a k-contiguous operand: pieces whose reduction index (k0: that of the slab) is >= K read zeros
  __device__ __forceinline__ void mask_beyond(int k0, int wave, int lane) {
    if constexpr (!KS) {
#pragma unroll
      for (int i = 0; i < N; ++i) {
        int row, piece;
        place_of(i, wave, lane, row, piece);
        voff[i] = k0 + piece * 8 < K ? voff[i] : kOffNone;
      }
    }
  }
  // descriptor of slab `slab`; every part of it scalar (a clamp on the vector unit would make the loads a loop over lanes)
  __device__ __forceinline__ void point(int slab) {
    long off = slab * step;
    if constexpr (TWO_SEG) off += slab >= seg_slabs ? seg_delta : 0L;
    uint32_t range = slab < nslabs ? (KS ? kRangeRows : kRangeAll) : 0u;
    if constexpr (KS && !GATHER) {
      int first = slab * BK;
      if constexpr (TWO_SEG) first -= slab >= seg_slabs ? seg_slabs * BK : 0;
      int left = scalar_min(BK, K - first);
      left = max(left, 0);
      if constexpr (TWO_SEG) left = slab < nslabs ? left : 0;
      range = static_cast<uint32_t>(left) * ld2;
    }
    rsrc = __builtin_amdgcn_make_buffer_rsrc(const_cast<char*>(base + off), 0, static_cast<int>(range), 0x00020000);
    if constexpr (KS && GATHER) {
      // byte offsets of the wave's rows; rows beyond K are beyond the range
#pragma unroll
      for (int j = 0; j < NR; ++j) next_row[j] = slab * BK + k_first + j < K ? static_cast<int32_t>(static_cast<uint32_t>(next_row[j]) * ld2) : static_cast<int32_t>(kRangeRows);
    }
  }
  // byte offset of this lane's piece of chunk i
  __device__ __forceinline__ uint32_t lane_off(int i) const {
    if constexpr (KS && GATHER) {
      int32_t moff = next_row[i * KPC];
#pragma unroll
      for (int q = 1; q < KPC; ++q) moff = lq == q ? next_row[i * KPC + q] : moff;
      return static_cast<uint32_t>(moff) + voff[i];
    } else {
      return voff[i];
    }
  }
  // one of the N loads of the slab that point() described, into the operand tile at `tile` (LDS); slabs are issued in order
  __device__ __forceinline__ void issue_at(int i, uint32_t off, char* tile, int wave) const {
    __builtin_amdgcn_raw_ptr_buffer_load_lds(rsrc, (__attribute__((address_space(3))) void*)(tile + (wave * N + i) * 1024), 16, static_cast<int>(off), 0, 0, 0);
  }
  __device__ __forceinline__ void issue_one(int i, char* tile, int wave) const { issue_at(i, lane_off(i), tile, wave); }
  // a whole slab, then the row list of the one after it
  __device__ __forceinline__ void issue(int slab, char* tile, int wave) {
    point(slab);
#pragma unroll
    for (int i = 0; i < N; ++i) issue_one(i, tile, wave);
    fetch_rows(slab + 1);
  }
};

// s_waitcnt that waits only for the vector-memory counter to drop to n (gfx9 encoding:
// vmcnt = imm[3:0] | imm[15:14] << 4, expcnt = imm[6:4], lgkmcnt = imm[11:8])
template <int n> __device__ __forceinline__ void wait_vmcnt() {
  __builtin_amdgcn_s_waitcnt((n & 15) | (7 << 4) | (15 << 8) | ((n >> 4) << 14));
}

// a wave's accumulators
template <class T> using Acc = f32x4[T::FM][T::FN];
template <class T>
__device__ __forceinline__ void zero_acc(Acc<T>& acc) {
#pragma unroll
  for (int i = 0; i < T::FM; ++i)
#pragma unroll
    for (int j = 0; j < T::FN; ++j)
#pragma unroll
      for (int q = 0; q < 4; ++q) acc[i][j][q] = 0.0f;
}

// acc += sum over segments of A_s(BM x K) * B_s(BN x K)^T for this wave's sub-tile (segments differ
// only in their base pointers).
//
// The MFMA is the 16 x 16 x 32 one: kept busy, it does 13-17 % more arithmetic per second on random operands than the
// 32 x 32 x 16 one (256 CUs, operands in registers: 1974-2128 against 1713-1880 TFLOP/s; with the LDS reads of a
// 128 x 64 sub-tile 1768-1851 against 1680-1694: in both the clock falls below its 2.4 GHz).
//
// What bounds the loop (stamps of a build with one tile per workgroup): a slab of the gate/up product at 2560 rows per expert takes 2.62 k clocks at 1.86 GHz = 1.41 us
// (64 MFMAs per wave, two waves per SIMD: 2.05 k clocks).  The loads and barriers alone take 1.36 us (at 2.39 GHz), the
// MFMAs and LDS reads alone 1.10 us (at 2.06 GHz): the row products run at the rate the slabs arrive, 64 KiB per CU, which is a
// matter of latency (the same loads without barriers, 32 KiB per CU in flight: 0.5-0.65 us) and hardly of the clock, which falls with the load.
// So what leaves the slabs' arrival as it is leaves the time as it is: four waves of 128 x 128 per tile, with two thirds of the LDS reads, take the
// same time a slab (and twice as long in the epilogues: 0.97 of the speed), and a tenth less read from memory changes little (see kGroup).  The
// weight gradients' loads alone take 1.12-1.21 us, their MFMAs and LDS reads 1.25 us, together 1.60 us at 1.70-1.76 GHz.
//
// Slabs stream through the two LDS rings (SA buffers for the A side, SB for the B side) filled by direct
// global->LDS loads.  A slab is two reduction steps (S0, S1) of FM rows of FN MFMAs.  A row-side fragment is read again
// for the next step right after the last MFMA that consumes it, so it has the FM - 1 other rows to arrive; the
// column-side fragments, which every row uses, are double-buffered in registers.  Per slab kt:
//     S0: row i | read a_i of S1, then b_j of S1 | (spread) refill B of slab kt+SB-1, whose buffer slab kt-1 has left
//     S1: rows 0 .. R0-1
//         wait: own LDS reads of slab kt complete, own loads of slab kt+1 landed (later slabs stay in flight)
//         barrier: slab kt+1 is visible to all, and nobody reads the buffers of slab kt any more
//         read b, a_0 .. a_R0-1 of S0 of slab kt+1
//         refill A of slab kt+SA, at once
//         rows R0 .. | read a_i of S0 of slab kt+1
// LDS reads of a wave complete in order, so "fragment X has arrived" is a wait for all but the reads issued after it;
// loads complete in the order they were enqueued, so "slab kt+1 has landed" is a wait for all but the loads enqueued
// after it -- immediates, both.
// Behind the last slabs of a tile come the first of the workgroup's next one, or empty slabs if there is none.  With one tile per
// workgroup 5.4-6.8 k clocks passed from a workgroup's entry to its first slab, and 3.4 us from the last store of a workgroup to the
// entry of the next.  Down, dX and the weight gradients keep slabs in flight from tile to tile.  Loads into registers are
// awaited with everything older, so where a product reads data of its rows the rings drain for a moment: for the gathered row list two slabs
// before a tile's end, for gate/up's combine weights at a tile's first slab and in its epilogue, for dA's G and U in the epilogue.
// At T = 8192, E = 128, k = 8, d = 2048, f = 768, one tile per workgroup -> several, timed in turn: weight gradients 747 -> 671 us, down 242 ->
// 229, gate/up 433 -> 434, dA 263 -> 268, dX 407 -> 421, the six products 2091 -> 2022.  (dA's epilogue takes 16 rows at a time in one
// buffer where it had 32 in the whole LDS; the row products' reads from memory grew, dX's by 11 %.)
// The loop is a plain loop over one slab body with run-time ring positions, a single path: with a body chosen per slab
// the compiler keeps fragments and accumulators in scratch memory.  The address registers of the fragments are
// advanced once per slab (4 to 12 vector additions against 64 MFMAs).
template <class T, bool A_KS, bool B_KS, bool A_GATHER = false, bool B_GATHER = false, int B_HALF = T::WN / 2, bool TWO_SEG = false>
struct MainLoop {
  typedef Dma<A_KS, T::BM, T::BK, T::kWaves, A_GATHER, TWO_SEG> DmaA;
  typedef Dma<B_KS, T::BN, T::BK, T::kWaves, B_GATHER, TWO_SEG> DmaB;
  static constexpr int NA = DmaA::N, NB = DmaB::N;     // loads per thread per slab and side
  static constexpr int SA = T::SA, SB = T::SB;
  static constexpr int FM = T::FM, FN = T::FN;
  static_assert(SA == 2 && SB == 3, "slab kt+2 is enqueued while slab kt is multiplied, on the row side after its barrier");
  static constexpr int kAhead = 2;                     // slabs in the rings when one is begun
  static constexpr int STEPS = T::BK / 32;
  static_assert(STEPS == 2, "a slab is two reduction steps");
  static constexpr int R0 = FM >= 8 ? 2 : 1;           // rows of S1 before the barrier
  static_assert(FM > R0, "rows of S1 after the barrier");
  static_assert((SA - 1) * NA + (SB - 1) * NB < 64, "vmcnt is a 6-bit counter");
  static constexpr int RA = A_KS ? 2 : 1, RB = B_KS ? 2 : 1;   // LDS instructions per fragment

  DmaA da;
  DmaB db;
  // Per-lane LDS addresses of the fragments.  k-contiguous side: a fragment 16 rows further is a constant number of
  // bytes further (the swizzle of a row repeats every 16 rows), while the step moves the piece index by 4, an XOR of
  // the address: one register per step, [0] in the buffer of the NEXT slab (its S0 is what is read ahead), [1] in that of
  // the slab being multiplied.  k-strided side: the step is a constant number of bytes (32 reduction rows; their
  // swizzle is the same) but a fragment 16 columns further is not: one register per fragment, moved on to the next
  // slab's buffer after its S1 read.
  static constexpr int NAA = A_KS ? FM : STEPS, NAB = B_KS ? FN : STEPS;
  uint32_t aa[NAA], ab[NAB];
  // Column-side fragments: two sets (S0, S1), or with four waves per SIMD -- 128 registers each, and three other waves to
  // cover an LDS latency -- one, each fragment read again right after its last MFMA, in the last row of the step.
  static constexpr bool B_ROLL = T::kWavesPerSimd >= 4;
  bf16x8 a[FM];
  bf16x8 b[B_ROLL ? 1 : 2][FN];
  static constexpr int b_set(int kk) { return B_ROLL ? 0 : kk; }
  char* lds;
  uint32_t lds32;                                      // the ring's start as an LDS address
  int stage_a, stage_b;                                // ring positions of the slab being multiplied
  int wave;
  int ls;                                              // slab that is enqueued next, of the tile the loads point at

  // tile rows between the wave's first fragment of a side and fragment i (the second half of the column side may lie apart)
  static constexpr int a_frag_row(int i) { return 16 * i; }
  static constexpr int b_frag_row(int i) { return (i >= FN / 2 ? B_HALF : 0) + 16 * (i % (FN / 2)); }
  static __device__ __forceinline__ int next_stage(int s, int n) { return s + 1 == n ? 0 : s + 1; }
  __device__ __forceinline__ char* buf_a(int stage) const { return lds + stage * T::kABytes; }
  __device__ __forceinline__ char* buf_b(int stage) const { return lds + T::kBBase + stage * T::kBBytes; }

  // ---- LDS reads of reduction step KK ----
  template <int KK, int I> __device__ __forceinline__ void read_a() {
    if constexpr (A_KS) a[I] = lds_read_frag<true, T::BM, KK * 32 * T::BM * 2>(aa[I]);
    else a[I] = lds_read_frag<false, T::BM, a_frag_row(I) * T::BK * 2>(aa[KK]);
  }
  template <int KK, int J> __device__ __forceinline__ void read_b() {
    if constexpr (B_KS) b[b_set(KK)][J] = lds_read_frag<true, T::BN, KK * 32 * T::BN * 2>(ab[J]);
    else b[b_set(KK)][J] = lds_read_frag<false, T::BN, b_frag_row(J) * T::BK * 2>(ab[KK]);
  }
  template <int KK, int J, int JEND> __device__ __forceinline__ void read_range_b() {
    if constexpr (J < JEND) { read_b<KK, J>(); read_range_b<KK, J + 1, JEND>(); }
  }
  template <int KK, int I, int IEND> __device__ __forceinline__ void read_range_a() {
    if constexpr (I < IEND) { read_a<KK, I>(); read_range_a<KK, I + 1, IEND>(); }
  }
  // Wait until at most N of this wave's LDS reads are outstanding (the counter has 4 bits: more is the same as 15), with
  // the fragments that have arrived by then as operands of the wait: the registers an asynchronous read is filling stay
  // reserved until here on every path -- the compiler must neither reuse them earlier nor move a consumer above the wait.
  template <int N> static __device__ __forceinline__ void arrived(bf16x8& x) {
    asm volatile("s_waitcnt lgkmcnt(%1)" : "+v"(x) : "n"(N < 15 ? N : 15));
  }
  template <int N, int KK> __device__ __forceinline__ void arrived_with_b(bf16x8& x) {
    static_assert(FN == 4, "add the operand list of this wave shape");
    constexpr int Q = b_set(KK);
    asm volatile("s_waitcnt lgkmcnt(%5)" : "+v"(x), "+v"(b[Q][0]), "+v"(b[Q][1]), "+v"(b[Q][2]), "+v"(b[Q][3]) : "n"(N < 15 ? N : 15));
  }
  __device__ __forceinline__ void all_arrived() {      // every row-side fragment
    static_assert(FM == 2 || FM == 4 || FM == 8, "add the operand list of this wave shape");
    if constexpr (FM == 8)
      asm volatile("s_waitcnt lgkmcnt(0)" : "+v"(a[0]), "+v"(a[1]), "+v"(a[2]), "+v"(a[3]), "+v"(a[4]), "+v"(a[5]), "+v"(a[6]), "+v"(a[7]));
    else if constexpr (FM == 4)
      asm volatile("s_waitcnt lgkmcnt(0)" : "+v"(a[0]), "+v"(a[1]), "+v"(a[2]), "+v"(a[3]));
    else
      asm volatile("s_waitcnt lgkmcnt(0)" : "+v"(a[0]), "+v"(a[1]));
  }
  // the MFMAs of one row of a step
  template <int KK, int I> __device__ __forceinline__ void mma_row(Acc<T>& acc) {
#pragma unroll
    for (int j = 0; j < FN; ++j)
      acc[I][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(b[b_set(KK)][j], a[I], acc[I][j], 0, 0, 0);   // transposed tile, see Strip
  }
  // the same for the last row of a step with B_ROLL: each column-side fragment is read for step NKK once it is free
  template <int KK, int NKK, int J = 0> __device__ __forceinline__ void mma_row_roll(int adv_b, Acc<T>& acc) {
    if constexpr (J < FN) {
      acc[FM - 1][J] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(b[0][J], a[FM - 1], acc[FM - 1][J], 0, 0, 0);
      __builtin_amdgcn_sched_barrier(0);
      read_b<NKK, J>();
      if constexpr (B_KS && NKK == 1) ab[J] += adv_b;
      __builtin_amdgcn_sched_barrier(0);
      mma_row_roll<KK, NKK, J + 1>(adv_b, acc);
    }
  }

  // ---- refill ----
  // The B side has nearly two slab periods from its refill to its use: its loads are spread over the rows of S0.  The A
  // side has one: it is enqueued right after the barrier, where it is not held up by MFMAs that a wave of the lower priority
  // on its SIMD has to wait for (spread over the rows of S1 instead, at 2560 rows per expert: gate/up 4.6 % slower, down
  // 3.5 %, dX 3.9 %).
  static constexpr int load_at(int n, int row) { return n * row / FM; }
  template <int J, int JEND> __device__ __forceinline__ void refill_a(char* tile) {
    if constexpr (J < JEND) { da.issue_one(J, tile, wave); refill_a<J + 1, JEND>(tile); }
  }
  template <int J, int JEND> __device__ __forceinline__ void refill_b(char* tile) {
    if constexpr (J < JEND) { db.issue_one(J, tile, wave); refill_b<J + 1, JEND>(tile); }
  }

  // column-side fragments of S1 read before row `row` of S0 (as early as the rows allow)
  static constexpr int kBPerRow = 2 * FN > FM ? 2 * FN / FM : 1;
  static constexpr int b_at(int row) { return B_ROLL ? 0 : row * kBPerRow < FN ? row * kBPerRow : FN; }
  static constexpr int last_b_row() { int r = 0; while (!B_ROLL && b_at(r + 1) < FN) ++r; return r; }
  // rows I .. of S0
  template <int I>
  __device__ __forceinline__ void step0(char* new_b, int adv_a, int adv_b, Acc<T>& acc) {
    if constexpr (I < FM) {
      // B_ROLL: the last row-side read follows those of the column side; row 0 has waited for all but it
      constexpr int YOUNGER = B_ROLL ? (I == FM - 1 ? FM - 1 : I + 1) * RA : (FM - 1 - I) * RA + I * RA + b_at(I) * RB;
      if constexpr (I == 0) arrived_with_b<YOUNGER, 0>(a[0]);
      else arrived<YOUNGER>(a[I]);
      __builtin_amdgcn_sched_barrier(0);
      if constexpr (B_ROLL && I == FM - 1) mma_row_roll<0, 1>(adv_b, acc);
      else mma_row<0, I>(acc);
      __builtin_amdgcn_sched_barrier(0);
      read_a<1, I>();
      if constexpr (A_KS) aa[I] += adv_a;
      read_range_b<1, b_at(I), b_at(I + 1)>();
      if constexpr (B_KS) {
#pragma unroll
        for (int j = b_at(I); j < b_at(I + 1); ++j) ab[j] += adv_b;
      }
      refill_b<load_at(NB, I), load_at(NB, I + 1)>(new_b);
      __builtin_amdgcn_sched_barrier(0);
      step0<I + 1>(new_b, adv_a, adv_b, acc);
    }
  }
  // rows I .. R0-1 of S1, before the barrier
  template <int I>
  __device__ __forceinline__ void step1_head(Acc<T>& acc) {
    if constexpr (I < R0) {
      // younger than a_I and every b of S1: the row-side reads issued after the later of them
      constexpr int FROM = I > last_b_row() ? I : last_b_row(), YOUNGER = B_ROLL ? RA : (FM - 1 - FROM) * RA;
      if constexpr (I == 0) arrived_with_b<YOUNGER, 1>(a[0]);
      else arrived<YOUNGER>(a[I]);
      __builtin_amdgcn_sched_barrier(0);
      mma_row<1, I>(acc);
      __builtin_amdgcn_sched_barrier(0);
      step1_head<I + 1>(acc);
    }
  }
  // the other rows of S1; the first step of the next slab is read between them
  template <int I>
  __device__ __forceinline__ void step1_tail(Acc<T>& acc) {
    if constexpr (I < FM) {
      if constexpr (B_ROLL && I == FM - 1) mma_row_roll<1, 0>(0, acc);
      else mma_row<1, I>(acc);
      __builtin_amdgcn_sched_barrier(0);
      read_a<0, I>();
      __builtin_amdgcn_sched_barrier(0);
      step1_tail<I + 1>(acc);
    }
  }
  // A slab of a wave with rows.  On entry the reads of its S0 are in flight, on exit those of the slab that follows in the
  // rings -- after a tile's last one, of the next tile, which reads them again: a body of its own for the last slab costs
  // registers across the loop.
  __device__ __forceinline__ void slab(Acc<T>& acc) {
    const int na = next_stage(stage_a, SA), nb = next_stage(stage_b, SB);
    const int adv_a = (na - stage_a) * T::kABytes, adv_b = (nb - stage_b) * T::kBBytes;
    db.point(ls);
    step0<0>(buf_b(stage_b == 0 ? SB - 1 : stage_b - 1), adv_a, adv_b, acc);
    db.fetch_rows(ls + 1);
    step1_head<0>(acc);
    all_arrived();                                     // this wave no longer needs the buffers of slab kt
    wait_vmcnt<NB>();                                  // slab kt+1 has landed
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_sched_barrier(0);
    da.point(ls);
    if constexpr (!B_ROLL) read_range_b<0, 0, FN>();
    read_range_a<0, 0, R0>();
    __builtin_amdgcn_sched_barrier(0);
    refill_a<0, NA>(buf_a(stage_a));
    __builtin_amdgcn_sched_barrier(0);
    step1_tail<R0>(acc);
    da.fetch_rows(ls + 1);
    if constexpr (!A_KS) {
      aa[0] += (next_stage(na, SA) - na) * T::kABytes;
      aa[1] += adv_a;
    }
    if constexpr (!B_KS) {
      ab[0] += (next_stage(nb, SB) - nb) * T::kBBytes;
      ab[1] += adv_b;
    }
    __builtin_amdgcn_sched_barrier(0);
  }
  // the same of a wave without rows
  __device__ __forceinline__ void idle_slab() {
    db.issue(ls, buf_b(stage_b == 0 ? SB - 1 : stage_b - 1), wave);
    wait_vmcnt<NB>();
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_sched_barrier(0);
    da.issue(ls, buf_a(stage_a), wave);
  }

  // the first step of the slab at the rings' current positions
  __device__ __forceinline__ void read_first() {
    if constexpr (B_ROLL) {                            // in the order of the slab body
      read_range_a<0, 0, FM - 1>();
      read_range_b<0, 0, FN>();
      read_range_a<0, FM - 1, FM>();
    } else {
      read_range_b<0, 0, FN>();
      read_range_a<0, 0, FM>();
    }
    if constexpr (!A_KS) aa[0] += (next_stage(stage_a, SA) - stage_a) * T::kABytes;   // from here on [0] addresses the buffer of the next slab
    if constexpr (!B_KS) ab[0] += (next_stage(stage_b, SB) - stage_b) * T::kBBytes;
    __builtin_amdgcn_sched_barrier(0);
  }

  __device__ __forceinline__ void prepare(char* lds_) {
    wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);   // wave-uniform: LDS destinations stay scalar
    lds = lds_;
    lds32 = static_cast<uint32_t>(reinterpret_cast<uintptr_t>((__attribute__((address_space(3))) char*)lds_));
    stage_a = 0; stage_b = 0;
  }
  // fragment addresses at the rings' current positions (first tile rows of this wave's sub-tile: a_row / b_row)
  __device__ __forceinline__ void place(int a_row, int b_row, int lane) {
    const uint32_t at_a = lds32 + stage_a * T::kABytes, at_b = lds32 + T::kBBase + stage_b * T::kBBytes;
#pragma unroll
    for (int i = 0; i < NAA; ++i) {                    // k-strided: fragment i at step 0; k-contiguous: fragment 0 at step i
      if constexpr (A_KS) aa[i] = at_a + frag_off<true, T::BM, T::BK>(a_row + a_frag_row(i), 0, lane);
      else aa[i] = at_a + frag_off<false, T::BM, T::BK>(a_row, i, lane);
    }
#pragma unroll
    for (int i = 0; i < NAB; ++i) {
      if constexpr (B_KS) ab[i] = at_b + frag_off<true, T::BN, T::BK>(b_row + b_frag_row(i), 0, lane);
      else ab[i] = at_b + frag_off<false, T::BN, T::BK>(b_row, i, lane);
    }
  }

  // ---- tiles ----
  // Slabs of a tile: a reduction of K indices (TWO_SEG: twice), a partial last slab counted whole, at least kAhead (the rings
  // hold slabs of at most two tiles).
  static __device__ __forceinline__ int slabs_of(int K) { return (TWO_SEG ? 2 : 1) * ((K + T::BK - 1) / T::BK); }
  static __device__ __forceinline__ int slabs_run(int K) { return max(slabs_of(K), kAhead); }
  // Point the loads at a tile's operands.  K = 0: there is no such tile, and its slabs are empty.  TWO_SEG: two segments of K
  // indices each, columns 0 .. K-1 and K .. 2K-1 of the A side, opB and then opB2.
  __device__ __forceinline__ void load_tile(const Operand& opA, const Operand& opB, const bf16_t* b2, int K) {
    const int lane = not_before_here(threadIdx.x & 63), n = slabs_of(K);
    da.init(opA, K, n, wave, lane);
    db.init(opB, K, n, wave, lane);
    if constexpr (TWO_SEG) {
      static_assert(!TWO_SEG || (!A_KS && B_KS && !A_GATHER), "");
      da.seg_slabs = db.seg_slabs = n / 2;
      da.seg_delta = 2L * K - (n / 2) * da.step;
      db.seg_delta = reinterpret_cast<const char*>(b2) - reinterpret_cast<const char*>(opB.half[0]) - (n / 2) * db.step;
    }
    ls = 0;
  }
  // before slab `ls` is enqueued: a partial slab of a k-contiguous side
  __device__ __forceinline__ void before_slab() {
    if constexpr (!(A_KS && B_KS)) {
      if (da.K % T::BK != 0) {                         // (widths that are no multiple of 64)
        const int lane = not_before_here(threadIdx.x & 63);
        int s = ls;
        if constexpr (TWO_SEG) {
          if (s == da.seg_slabs) da.place_rows(wave, lane);
          if (s >= da.seg_slabs) s -= da.seg_slabs;
        }
        if (s == da.K / T::BK) {
          da.mask_beyond(s * T::BK, wave, lane);
          db.mask_beyond(s * T::BK, wave, lane);
        }
      }
    }
  }
  // the first kAhead slabs of the first tile into the idle rings; on return its first one has landed and is visible to all
  __device__ __forceinline__ void fill() {
#pragma unroll
    for (int s0 = 0; s0 < kAhead; ++s0) {
      before_slab();
      db.issue(ls, buf_b(s0), wave);
      da.issue(ls, buf_a(s0), wave);
      ++ls;
    }
    wait_vmcnt<NA + NB>();
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_sched_barrier(0);
  }
  // Multiply the n slabs of a tile, the first of which has landed at the rings' current positions; `next` points the loads
  // at the tile that follows, whose first kAhead slabs are enqueued behind this one's.
  // `active` is false for a wave whose sub-tile holds no row of the expert (the tile sticks out of the row segment): it
  // only takes part in the loads and barriers; its SIMD time goes to the other waves.
  template <bool ALWAYS_ACTIVE, class Next>
  __device__ __forceinline__ void tile(int n, int a_row, int b_row, bool active, Acc<T>& acc, const Next& next) {
    if (ALWAYS_ACTIVE || active) {
      place(a_row, b_row, not_before_here(threadIdx.x & 63));
      read_first();
    }
#pragma nounroll
    for (int kt = 0; kt < n; ++kt) {
      if (kt == n - kAhead) next();
      before_slab();
      if (ALWAYS_ACTIVE || active) slab(acc);
      else idle_slab();
      ++ls;
      stage_a = next_stage(stage_a, SA); stage_b = next_stage(stage_b, SB);
    }
    if (ALWAYS_ACTIVE || active) {
      all_arrived();                                   // nothing is in flight into a register when the epilogue starts
      arrived_with_b<0, 0>(a[0]);
    }
  }
  // After a tile: the part of the free column-side buffer that this wave's loads fill next (see the epilogue)
  static constexpr int kScratch = NB * 1024;
  __device__ __forceinline__ uint32_t scratch() const {
    return lds32 + T::kBBase + (stage_b == 0 ? SB - 1 : stage_b - 1) * T::kBBytes + wave * kScratch;
  }
  // the empty slabs behind the last tile write zeros into the LDS: they are awaited before the workgroup gives it back
  static __device__ __forceinline__ void finish() { wait_vmcnt<0>(); }
};

// ---- epilogue: accumulators -> LDS -> 16-byte row-contiguous global accesses -----------------------------
// The products are accumulated transposed (the MFMA is handed the weight-side fragment as its first operand): of the
// 16x16 tile (i, j) a lane then holds tile row lane%16 and the four consecutive columns 4*(lane/16) .. +3.  The memory
// pipeline joins the 16-byte accesses of four neighbouring lanes, so results pass through the LDS to give neighbouring lanes
// neighbouring columns (exchanged between lanes in registers, which gives them neighbouring rows, the stores of a
// 256 x 256 tile took 10k clocks instead of 5k).
//
// The rings hold the next tile's first two slabs by then, but one column-side buffer is free: the one that the next tile's
// slab 2 goes to.  A wave parks its results in the part of that buffer that its own loads will fill (kScratch bytes), so no
// other wave has to be waited for.  Parking writes and reads are assembly statements for the reason given at lds_read_frag;
// a wave's LDS accesses are executed in order, and every read is awaited inside its statement.
__device__ __forceinline__ void lds_park8(uint32_t addr, u32x2 v) { asm volatile("ds_write_b64 %0, %1" :: "v"(addr), "v"(v)); }
__device__ __forceinline__ void lds_park16(uint32_t addr, u32x4 v) { asm volatile("ds_write_b128 %0, %1" :: "v"(addr), "v"(v)); }
__device__ __forceinline__ void lds_fetch(uint32_t a0, uint32_t a1, u32x4& v0, u32x4& v1) {
  asm volatile("ds_read_b128 %0, %2\n\tds_read_b128 %1, %3\n\ts_waitcnt lgkmcnt(0)" : "=&v"(v0), "=&v"(v1) : "v"(a0), "v"(a1));
}
__device__ __forceinline__ void lds_fetch(uint32_t a0, uint32_t a1, uint32_t a2, uint32_t a3, u32x4& v0, u32x4& v1, u32x4& v2, u32x4& v3) {
  asm volatile("ds_read_b128 %0, %4\n\tds_read_b128 %1, %5\n\tds_read_b128 %2, %6\n\tds_read_b128 %3, %7\n\ts_waitcnt lgkmcnt(0)"
               : "=&v"(v0), "=&v"(v1), "=&v"(v2), "=&v"(v3) : "v"(a0), "v"(a1), "v"(a2), "v"(a3));
}
__device__ __forceinline__ u32x2 pack4(const f32x4& v) { return u32x2{pack_bf16x2(v[0], v[1]), pack_bf16x2(v[2], v[3])}; }

// 16 rows x 64 columns as bf16, 128 bytes per row; the 16-byte pieces of a row are XORed with the row.  fetch: lane l gets the
// columns 8 (l%8) .. +7 of row l/8 and of row 8 + l/8.
struct StripBf16 {
  uint32_t at_w, at_r;
  __device__ __forceinline__ StripBf16(uint32_t base, int lane) {
    const int r = lane & 15, q = lane >> 4, l3 = lane >> 3;
    at_w = base + r * 128 + (((q >> 1) ^ (r & 7)) << 4) + 8 * (q & 1);
    at_r = base + l3 * 128 + (((lane & 7) ^ l3) << 4);
  }
  __device__ __forceinline__ void park(int j, const f32x4& v) const { lds_park8(at_w ^ (j * 32), pack4(v)); }
  __device__ __forceinline__ void fetch(u32x4& lo, u32x4& hi) const { lds_fetch(at_r, at_r + 1024, lo, hi); }
};
// 16 rows x 64 columns of fp32, 256 bytes per row, swizzled likewise; fetch: as above, v[h] for row 8 h + l/8
struct StripF32 {
  uint32_t at_w, at_r;
  __device__ __forceinline__ StripF32(uint32_t base, int lane) {
    const int r = lane & 15, q = lane >> 4, l3 = lane >> 3;
    at_w = base + r * 256 + ((q ^ r) << 4);
    at_r = base + l3 * 256 + (((2 * (lane & 7)) ^ l3) << 4);
  }
  // (element by element: the compiler keeps vectors that are only used whole in one piece across the slab loop, and copies
  // of the accumulators in scratch memory)
  __device__ __forceinline__ void park(int j, const f32x4& v) const {
    u32x4 w;
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      float x = v[t];
      asm("" : "+v"(x));
      w[t] = __float_as_uint(x);
    }
    lds_park16(at_w ^ (j * 64), w);
  }
  __device__ __forceinline__ void fetch(float (&v)[2][8]) const {
    const uint32_t hi = (at_r ^ 128) + 2048;
    u32x4 a, b, c, d;
    lds_fetch(at_r, at_r ^ 16, hi, hi ^ 16, a, b, c, d);
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      v[0][q] = __uint_as_float(a[q]); v[0][4 + q] = __uint_as_float(b[q]);
      v[1][q] = __uint_as_float(c[q]); v[1][4 + q] = __uint_as_float(d[q]);
    }
  }
};

// sum over each aligned group of 8 consecutive lanes, left in every lane of the group; data-parallel primitives (register moves
// between lanes), fixed order of additions
__device__ __forceinline__ float sum_of_8_lanes(float v) {
  auto dpp = [](float x, auto ctrl) {
    return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, x), decltype(ctrl)::value, 0xF, 0xF, true));
  };
  v += dpp(v, std::integral_constant<int, 0xB1>{});          // quad_perm [1,0,3,2]
  v += dpp(v, std::integral_constant<int, 0x4E>{});          // quad_perm [2,3,0,1]
  v += dpp(v, std::integral_constant<int, 0x141>{});         // row_half_mirror: the other quad of the 8 lanes
  return v;
}

__device__ __forceinline__ void read8(const float* p, float (&v)[8]) {
  const float4 x = *reinterpret_cast<const float4*>(p), y = *reinterpret_cast<const float4*>(p + 4);
  v[0] = x.x; v[1] = x.y; v[2] = x.z; v[3] = x.w; v[4] = y.x; v[5] = y.y; v[6] = y.z; v[7] = y.w;
}
__device__ __forceinline__ u32x4 pack8(const float (&v)[8]) {
  return u32x4{pack_bf16x2(v[0], v[1]), pack_bf16x2(v[2], v[3]), pack_bf16x2(v[4], v[5]), pack_bf16x2(v[6], v[7])};
}
__device__ __forceinline__ void unpack8(const u32x4& w, float (&v)[8]) {
#pragma unroll
  for (int q = 0; q < 4; ++q) { v[2 * q] = bf16_lo(w[q]); v[2 * q + 1] = bf16_hi(w[q]); }
}

// Results are written once and read by a later kernel: a non-temporal store keeps them from displacing the
// operand panels that concurrently running tiles share through the L2 (measured: 2 % of the step).
__device__ __forceinline__ void store16(void* p, const u32x4& v) { __builtin_nontemporal_store(v, reinterpret_cast<u32x4*>(p)); }

// A few rows (of a strip or a tile) of a row-major matrix as a buffer: a load of a row or column that does not exist returns
// zeros and a store to it does nothing, so the epilogues need no branches and no 64-bit address arithmetic per access.
//   first: the first row at the tile's first column (uniform); rows: how many rows exist (any integer);
//   pitch: bytes per row; skip: bytes between the start of a row and the tile's first column
// Ranges and offsets have 32 bits, so a buffer spans no more rows than one wave takes: MAX = 32, and rows of up to 64 MiB lie
// below kNone; MAX = 64 (weight gradients), and rows below 64 MiB lie below kOffNone.
struct StripRows {
  __amdgpu_buffer_rsrc_t rsrc;
  static constexpr uint32_t kNone = 0x80000000u;       // offset of a column that does not exist (to which rows may be added)
  template <int MAX = 32> __device__ __forceinline__ void at(const void* first, int rows, uint32_t pitch, uint32_t skip) {
    int n = scalar(min(rows, MAX));
    n = max(n, 0);
    const uint32_t range = n > 0 ? static_cast<uint32_t>(n) * pitch - skip : 0u;
    rsrc = __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(first), 0, static_cast<int>(range), 0x00020000);
  }
  __device__ __forceinline__ void store(uint32_t off, const u32x4& v) const {          // non-temporal, as store16
    __builtin_amdgcn_raw_buffer_store_b128(v, rsrc, static_cast<int>(off), 0, 2);
  }
  template <bool CACHED> __device__ __forceinline__ void store_as(uint32_t off, const u32x4& v) const {
    __builtin_amdgcn_raw_buffer_store_b128(v, rsrc, static_cast<int>(off), 0, CACHED ? 0 : 2);
  }
  __device__ __forceinline__ void store(uint32_t off, float v) const {
    __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(unsigned int, v), rsrc, static_cast<int>(off), 0, 0);
  }
  __device__ __forceinline__ void store_byte(uint32_t off, uint32_t v) const {
    __builtin_amdgcn_raw_buffer_store_b8(static_cast<uint8_t>(v), rsrc, static_cast<int>(off), 0, 0);
  }
  __device__ __forceinline__ float load_float(uint32_t off) const {
    return __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(rsrc, static_cast<int>(off), 0, 0));
  }
  __device__ __forceinline__ u32x4 load(uint32_t off) const { return __builtin_amdgcn_raw_buffer_load_b128(rsrc, static_cast<int>(off), 0, 0); }
};

// ---- device-built schedule of (expert, row tile) for row-grouped products -----------------
struct RowTiles {
  int32_t* count;        // [1] number of row tiles
  TileEntry* entry;      // [max_tiles]
  int max_tiles;
  int bm;                // rows of a tile: which of the tile shapes the list is for
};

__device__ __forceinline__ void build_row_tiles(const int32_t* __restrict__ offsets, int E, int P, int bm, RowTiles rt) {
  __shared__ int32_t scan[kMaxExperts];     // inclusive scan of the row tiles per expert
  __shared__ int32_t first_row[kMaxExperts], end_row[kMaxExperts];
  const int e = threadIdx.x;
  int begin = 0, end = 0, nt = 0;
  if (e < E) {
    begin = min(max(offsets[e], 0), P);
    end = min(max(offsets[e + 1], begin), P);
    nt = (end - begin + bm - 1) / bm;
  }
  scan[e] = nt;
  first_row[e] = begin;
  end_row[e] = end;
  __syncthreads();
  for (int o = 1; o < 1024; o <<= 1) {
    int v = e >= o ? scan[e - o] : 0;
    __syncthreads();
    scan[e] += v;
    __syncthreads();
  }
  // offsets that are not a monotone scan ending at P cannot overflow the lists
  const int total = min(scan[1023], rt.max_tiles);
  // every thread writes the tiles t, t + 1024, ...
  for (int t = threadIdx.x; t < total; t += 1024) {
    const int x = expert_of_row_tile(scan, E, t);
    const TileEntry w = row_tile_entry(scan, x, t, total, first_row[x], end_row[x], bm);
    int4* const out = reinterpret_cast<int4*>(rt.entry + t);
    out[0] = int4{w.expert, w.first, w.n, w.row0};
    out[1] = int4{w.row_end, 0, 0, 0};
  }
  if (e == 1023) rt.count[0] = total;
}
__global__ __launch_bounds__(1024) void build_row_tiles_kernel(const int32_t* __restrict__ offsets, int E, int P,
                                                                int bm, RowTiles rt) {
  build_row_tiles(offsets, E, P, bm, rt);
}

// Lists that a launch only reads, as constant memory: uniform loads from them are scalar whatever the kernel has stored before.
typedef __attribute__((address_space(4))) const int32_t* ConstList;
__device__ __forceinline__ ConstList const_list(const int32_t* p) { return reinterpret_cast<ConstList>(reinterpret_cast<uintptr_t>(p)); }

// Tile v of a row-grouped product with n_tiles_n column tiles: its expert, rows and column tile n.
__device__ __forceinline__ TileAt tile_at(const RowTiles& rt, int v, int n_tiles_n, int bm) {
  typedef int32_t Words __attribute__((ext_vector_type(8), aligned(16)));   // (a workspace starts at a multiple of 16 bytes, not of 32)
  static_assert(sizeof(TileEntry) == sizeof(Words), "");
  const int mt = scalar(v / n_tiles_n);
  const Words w = *reinterpret_cast<__attribute__((address_space(4))) const Words*>(reinterpret_cast<uintptr_t>(rt.entry + mt));
  return tile_of_entry(TileEntry{w[0], w[1], w[2], w[3], w[4], {}}, v, n_tiles_n, bm, [](int x) { return scalar(x); });
}

// ============================================================================================
// Row-grouped kernels
// ============================================================================================

enum { kGateUp = 0, kDown = 1, kDAct = 2, kDX = 3, kRouterFwd = 4, kRouterDx = 5 };

struct RowArgs {
  const bf16_t* a;         // activation operand [P, lda]
  long lda;
  const bf16_t* w0;        // first weight  [E, ...]
  const bf16_t* w1;        // second weight (gate/up kinds) or null
  long w_expert_stride;    // elements between experts
  long ldw;                // row pitch of one expert's weight matrix
  int K;                   // reduction length per segment
  int N;                   // output columns
  int P;
  RowTiles rt;
  int n_tiles_n;
  bf16_t* out0;            // kGateUp: G (may be null)   kDown/kDX/kRouterDx: output     kDAct: [dG | dU]
  bf16_t* out1;            // kGateUp: U (may be null)
  bf16_t* out2;            // kGateUp: act (may be null)
  long ldo;
  float* out_f32;          // kRouterFwd: fp32 output
  int accumulate;          // kRouterDx: add to what out0 holds
  const bf16_t* g;         // kDAct: saved pre-activations
  const bf16_t* u;
  // FUSED kernels: `a` is the token-major matrix [T, lda] and row r of the product reads a[row_token[r]]
  const int32_t* row_token;    // [P (+ padding)]
  const float* row_w;          // kDAct: combine weight of each row; the product's rows are scaled by it
                               // kGateUp (may be null): the activation leaves scaled by it
  bf16_t* act_w;               // kDAct: [P, N] out, row_w * silu(G) * U; null: not written (the forward left it)
  float* dw_partial;           // kDAct: [n_tiles_n * WGN][P] out, partial sums of <silu(G) * U, unscaled dA> per row
};

// FUSED (kGateUp and kDAct only): the activation rows are gathered from the token-major matrix while the
// tiles are loaded, so no expert-ordered copy of it exists.  For kDAct that matrix is the gradient of the
// layer output, and the rest of the combine backward rides in the epilogue:
//   dA = w_r * (dy[token(r)] Wd)              the combine weight scales the product's rows
//   d w_r = <dy[token(r)], yp[r]> = <dy[token(r)] Wd, act[r]>    reduced over the columns of the tile
//   act_w[r] = w_r * act[r]                   the operand with which dWd = dy[token]^T act_w needs no dyp
// OPTION, kDAct: act_w is written (else the forward left it); kGateUp: its half-line stores go through the L2 (see launch_gate_up).
template <int KIND, class T, bool FUSED = false, bool OPTION = false>
__global__ __launch_bounds__(T::kThreads) __attribute__((amdgpu_waves_per_eu(T::kWavesPerSimd, T::kWavesPerSimd))) void row_grouped_kernel(RowArgs p) {
  static_assert(!FUSED || KIND == kGateUp || KIND == kDAct, "only the two products that read activations by token are fused");
  extern __shared__ __attribute__((aligned(16))) char lds[];
  constexpr int BM = T::BM, BN = T::BN, WM = T::WM, WN = T::WN, MI = T::MI, FN = T::FN;
  static_assert(FN == 4, "the epilogues take the fragments of a row in two pairs");
  constexpr bool B_STRIDED = KIND == kDAct || KIND == kRouterDx || KIND == kDX, TWO_SEG = KIND == kDX;
  // kGateUp: tile columns are BN/2 gate columns n0.. and the matching BN/2 up columns; each wave gets the same gate and up
  // columns (the up fragments lie BN/2 tile rows further), so a lane holds the gate and the up value of an output
  constexpr int HN = BN / 2, HW = WN / 2, OUT_N = KIND == kGateUp ? HN : BN;
  typedef MainLoop<T, false, B_STRIDED, FUSED, false, KIND == kGateUp ? HN : WN / 2, TWO_SEG> Loop;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int wm = wave / T::WGN, wn = wave % T::WGN;
  const int a_row = wm * WM, b_row = wn * (KIND == kGateUp ? HW : WN);   // first tile rows of this wave on either side

  // This workgroup's tiles: every gridDim.x-th of the list (see xcd_remap), the next one located while one is multiplied.
  // The router's products have one segment of all rows: its row tiles follow from their number.
  constexpr bool ONE_SEGMENT = KIND == kRouterFwd || KIND == kRouterDx;
  const int total = (ONE_SEGMENT ? (p.P + BM - 1) / BM : const_list(p.rt.count)[0]) * p.n_tiles_n;
  // (`exists` is a number of unknown origin: a truth value carried around the loop would be a lane mask, and the parts of the
  // descriptors that are selected by it vectors, which makes every load of the slab loop a loop over lanes)
  struct At { int row0, rows, e, n0, exists; };
  auto locate = [&](int block) {
    At t{};
    const int v = xcd_remap(block, total);
    t.exists = scalar(v >= 0 ? 1 : 0);
    if (v >= 0) {
      if constexpr (ONE_SEGMENT) {
        const int mt = scalar(v / p.n_tiles_n);
        t.n0 = (v - mt * p.n_tiles_n) * OUT_N;
        t.row0 = mt * BM;
        t.rows = scalar(min(BM, p.P - t.row0));
      } else {
        const TileAt at = tile_at(p.rt, v, p.n_tiles_n, BM);
        t.e = at.e; t.row0 = at.row0; t.rows = at.rows;
        t.n0 = at.n * OUT_N;
      }
    }
    return t;
  };
  int block = blockIdx.x;
  At cur = locate(block);
  if (cur.exists == 0) return;

  Loop ml;
  auto load = [&](const At& t) {
    Operand opA, opB;
    opA.ld = p.lda;
    opA.valid[0] = min(t.rows, BM / 2);
    opA.valid[1] = max(t.rows - BM / 2, 0);
    opA.half[0] = FUSED ? p.a : p.a + static_cast<long>(t.row0) * p.lda;
    opA.half[1] = FUSED ? p.a : opA.half[0] + (BM / 2) * p.lda;
    opA.gather = FUSED ? p.row_token : nullptr;
    opA.grow = t.row0;
    opB.ld = p.ldw;
    opB.gather = nullptr;
    opB.grow = 0;
    const int ncols = scalar(min(OUT_N, p.N - t.n0));
    const bf16_t* w0 = p.w0 + t.e * p.w_expert_stride;
    const bf16_t* w1 = nullptr;
    if constexpr (KIND == kGateUp) {
      opB.half[0] = w0 + static_cast<long>(t.n0) * p.ldw;
      opB.half[1] = p.w1 + t.e * p.w_expert_stride + static_cast<long>(t.n0) * p.ldw;
      opB.valid[0] = opB.valid[1] = ncols;
    } else {
      opB.valid[0] = min(ncols, BN / 2);
      opB.valid[1] = max(ncols - BN / 2, 0);
      // yp = act * Wd[e]^T (logits = x * Wr^T): weight rows are output columns, reduction contiguous
      // dA = dyp * Wd[e] (dx = dz * Wr), dxp = dG * Wg[e] + dU * Wu[e]: weight is [K, N], reduction strided
      opB.half[0] = B_STRIDED ? w0 + t.n0 : w0 + static_cast<long>(t.n0) * p.ldw;
      opB.half[1] = B_STRIDED ? opB.half[0] + BN / 2 : opB.half[0] + (BN / 2) * p.ldw;
      if constexpr (TWO_SEG) w1 = p.w1 + t.e * p.w_expert_stride + t.n0;
    }
    ml.load_tile(opA, opB, w1, p.K * t.exists);
  };
  ml.prepare(lds);
  load(cur);
  ml.fill();
  const int n_slabs = Loop::slabs_run(p.K);

  for (;;) {
    block += gridDim.x;
    const At nxt = locate(block);
    const int rows = cur.rows, row0 = cur.row0, n0 = cur.n0;
    const int ncols = min(OUT_N, p.N - n0);
    // 32-row strips of this wave that hold rows of the expert (wave-uniform); a wave without any
    // skips the arithmetic, and the epilogue skips strips without rows (its origin hidden: a compiler that knows where it comes
    // from splits the paths behind the main loop by its value and spills the accumulators on them)
    const int mi_n = scalar(min(MI, max(0, (rows - a_row + 31) / 32)));
    // the combine weights of the wave's rows: lane l holds those of rows l, l + 64, ...
    constexpr int NW = KIND == kGateUp ? (WM + 63) / 64 : 1;
    float row_w[NW];
    if constexpr (KIND == kGateUp) {
#pragma unroll
      for (int c = 0; c < NW; ++c) {
        const int r = a_row + c * 64 + lane;
        row_w[c] = p.row_w ? p.row_w[row0 + (r < rows ? r : 0)] : 1.0f;
      }
    }
    Acc<T> acc;
    zero_acc<T>(acc);
    ml.template tile<false>(n_slabs, a_row, b_row, mi_n > 0, acc, [&] { load(nxt); });

    const int el = not_before_here(lane);              // this lane, for the epilogue
    const uint32_t scratch = ml.scratch();
    static_assert(Loop::kScratch >= (KIND == kDown || KIND == kDX ? 2048 : KIND == kGateUp ? 3072 : 4096), "strips of 16 rows");
    auto weight_of = [&](int r) {                      // combine weight of the wave's row r (per lane, r - r%16 uniform)
      return __builtin_bit_cast(float, __builtin_amdgcn_ds_bpermute((r & 63) * 4, __builtin_bit_cast(int, r < 64 ? row_w[0] : row_w[NW - 1])));
    };
    const uint32_t ld2 = static_cast<uint32_t>(p.ldo) * 2u, skip2 = static_cast<uint32_t>(n0) * 2u;
    const int cl = b_row + 8 * (el & 7), rl = el >> 3; // row-major: this lane's 8 columns, and its row in each 8 rows
    auto off8 = [&](uint32_t pitch) { return off_if(cl < ncols, rl * pitch + cl * 2u, StripRows::kNone); };
    if constexpr (KIND == kGateUp) {
      // 16 rows x (32 gate + 32 up columns) parked as they are, 16 x 32 activations behind them; 4 lanes per row of 64 bytes
      const int r = el & 15, q = el >> 4, r4 = el >> 2, c4 = el & 3;
      const StripBf16 gu(scratch, el);
      const uint32_t gu_r = scratch + r4 * 128 + ((c4 ^ (r4 & 7)) << 4);
      const uint32_t act_w = scratch + 2048 + r * 64 + (((q >> 1) ^ ((r >> 1) & 3)) << 4) + 8 * (q & 1), act_r = scratch + 2048 + r4 * 64 + ((c4 ^ ((r4 >> 1) & 3)) << 4);
      const int col = b_row + 8 * c4;
      const uint32_t off = off_if(col < ncols, r4 * ld2 + col * 2u, StripRows::kNone);
#pragma unroll
      for (int mi = 0; mi < MI; ++mi) {
        if (mi >= mi_n) break;
#pragma unroll
        for (int h = 0; h < 2; ++h) {
          const int i = 2 * mi + h, rs0 = a_row + i * 16;   // first row of the strip inside the tile
          const float w = weight_of(i * 16 + r);
#pragma unroll
          for (int j = 0; j < FN; ++j) gu.park(j, acc[i][j]);
#pragma unroll
          for (int j = 0; j < 2; ++j) {
            f32x4 a;
#pragma unroll
            for (int t = 0; t < 4; ++t) a[t] = w * (acc[i][j][t] * sigmoid_fast(acc[i][j][t]) * acc[i][j + 2][t]);
            lds_park8(act_w ^ (j * 32), pack4(a));
          }
          u32x4 vg, vu, va, unused;
          lds_fetch(gu_r, gu_r ^ 64, act_r, act_r, vg, vu, va, unused);
          const long o = static_cast<long>(row0 + rs0) * p.ldo + n0;
          StripRows sg, su, sa;
          sg.at(p.out0 + o, p.out0 ? rows - rs0 : 0, ld2, skip2);
          su.at(p.out1 + o, p.out1 ? rows - rs0 : 0, ld2, skip2);
          sa.at(p.out2 + o, p.out2 ? rows - rs0 : 0, ld2, skip2);
          sg.template store_as<OPTION>(off, vg);
          su.template store_as<OPTION>(off, vu);
          sa.template store_as<OPTION>(off, va);
        }
      }
    } else if constexpr (KIND == kDown || KIND == kDX) {
      const StripBf16 strip(scratch, el);
      const uint32_t off = off8(ld2);
#pragma unroll
      for (int mi = 0; mi < MI; ++mi) {
        if (mi >= mi_n) break;
        const int rs0 = a_row + mi * 32;
        StripRows so;
        so.at(p.out0 + static_cast<long>(row0 + rs0) * p.ldo + n0, rows - rs0, ld2, skip2);
#pragma unroll
        for (int h = 0; h < 2; ++h) {
#pragma unroll
          for (int j = 0; j < FN; ++j) strip.park(j, acc[2 * mi + h][j]);
          u32x4 v[2];
          strip.fetch(v[0], v[1]);
#pragma unroll
          for (int c = 0; c < 2; ++c) so.store(off + (16 * h + 8 * c) * ld2, v[c]);
        }
      }
    } else if constexpr (KIND == kDAct) {
      // The saved G and U of 16 rows are requested 16 rows ahead (the fragment registers are free now), and with them the rows'
      // combine weights: held across the slab loop, those made the 256 x 256 tile reload registers from scratch memory for every
      // tile (4096 tokens on 16 experts 81 -> 80 us, 8192 on 128 270 -> 268, 1531 107 -> 105).  This epilogue is
      // bound by the vector unit: 128 derivatives per lane, about 25 issue slots each, two waves per SIMD; it takes 24k of
      // the 111k clocks of a tile (2560 rows per expert).
      const StripF32 strip(scratch, el);
      const uint32_t n2 = static_cast<uint32_t>(p.N) * 2u;
      const uint32_t off = off8(ld2), goff = off8(n2);
      u32x4 gq[2][2], uq[2][2];                        // [fragment & 1][rows 0..7, 8..15]
      float wq[2][2];
      auto request = [&](int i) {
        const int rs0 = a_row + i * 16;
        const long gi = static_cast<long>(row0 + rs0) * p.N + n0;
        StripRows sg, su;
        sg.at(p.g + gi, rows - rs0, n2, skip2);
        su.at(p.u + gi, rows - rs0, n2, skip2);
#pragma unroll
        for (int c = 0; c < 2; ++c) {
          gq[i & 1][c] = sg.load(goff + 8 * c * n2);
          uq[i & 1][c] = su.load(goff + 8 * c * n2);
        }
        if constexpr (FUSED) {
          StripRows sw;
          sw.at(p.row_w + row0 + rs0, rows - rs0, 4, 0);
#pragma unroll
          for (int c = 0; c < 2; ++c) wq[i & 1][c] = sw.load_float((8 * c + rl) * 4u);
        }
      };
      request(0);
#pragma unroll
      for (int mi = 0; mi < MI; ++mi) {
        if (mi >= mi_n) break;
        const int rs0 = a_row + mi * 32;
        StripRows sd, saw, sdw;                          // (a row of [dG | dU] is one: dU lies n2 bytes further in it)
        sd.at(p.out0 + static_cast<long>(row0 + rs0) * p.ldo + n0, rows - rs0, ld2, skip2);
        if constexpr (FUSED) {
          if constexpr (OPTION) saw.at(p.act_w + (static_cast<long>(row0 + rs0) * p.N + n0), rows - rs0, n2, skip2);
          sdw.at(p.dw_partial + static_cast<long>(n0 / BN * T::WGN + wn) * p.P + row0 + rs0, min(rows - rs0, 32), 4, 0);
        }
#pragma unroll
        for (int h = 0; h < 2; ++h) {
          const int i = 2 * mi + h;
          if (i + 1 < T::FM) request(i + 1);
#pragma unroll
          for (int j = 0; j < FN; ++j) strip.park(j, acc[i][j]);
          float v[2][8];
          strip.fetch(v);
#pragma unroll
          for (int c = 0; c < 2; ++c) {
            float g[8], u[8], dg[8], du[8];
            unpack8(gq[i & 1][c], g);
            unpack8(uq[i & 1][c], u);
            const uint32_t down = (16 * h + 8 * c);      // rows below the strip's first
            // silu'(g) = sg (1 + g (1 - sg)) = sg + t (1 - sg) with t = g sg = silu(g); 1 - sg is formed first: where it is zero
            // the result is sg however large t is (sg + t - t sg would lose sg)
            if constexpr (FUSED) {
              const float w = wq[i & 1][c];
              float part = 0.0f, act[8];
#pragma unroll
              for (int q = 0; q < 8; ++q) {
                const float sg = sigmoid_fast(g[q]), t = g[q] * sg, da = w * v[c][q];
                act[q] = t * u[q];
                part = fmaf(act[q], v[c][q], part);
                dg[q] = (da * u[q]) * fmaf(t, 1.0f - sg, sg);
                du[q] = da * t;
              }
              sd.store(off + down * ld2, pack8(dg));
              sd.store(off + down * ld2 + n2, pack8(du));
              if constexpr (OPTION) {
#pragma unroll
                for (int q = 0; q < 8; ++q) act[q] *= w;
                saw.store(goff + down * n2, pack8(act));
              }
              // the 8 lanes of a row add up their columns (one that does not exist holds NaN if the row of dy has an
              // infinity); every (column slot, row) is written exactly once
              part = sum_of_8_lanes(cl < ncols ? part : 0.0f);
              sdw.store(off_if((el & 7) == 0, (down + rl) * 4u, StripRows::kNone), part);
            } else {
#pragma unroll
              for (int q = 0; q < 8; ++q) {
                const float sg = sigmoid_fast(g[q]), t = g[q] * sg;
                dg[q] = (v[c][q] * u[q]) * fmaf(t, 1.0f - sg, sg);
                du[q] = v[c][q] * t;
              }
              sd.store(off + down * ld2, pack8(dg));
              sd.store(off + down * ld2 + n2, pack8(du));
            }
          }
        }
      }
    } else {                                           // the router's
      const StripF32 strip(scratch, el);
#pragma unroll
      for (int i = 0; i < T::FM; ++i) {
        if (i >= 2 * mi_n) break;
        const int rs0 = a_row + i * 16;
#pragma unroll
        for (int j = 0; j < FN; ++j) strip.park(j, acc[i][j]);
        float v[2][8];
        strip.fetch(v);
        StripRows so;
        if constexpr (KIND == kRouterFwd) {
          const uint32_t ld4 = static_cast<uint32_t>(p.ldo) * 4u;
          so.at(p.out_f32 + static_cast<long>(row0 + rs0) * p.ldo + n0, rows - rs0, ld4, n0 * 4u);
          const uint32_t off = off_if(cl < ncols, rl * ld4 + cl * 4u, StripRows::kNone);
#pragma unroll
          for (int c = 0; c < 2; ++c)
#pragma unroll
            for (int t = 0; t < 2; ++t) {
              u32x4 o;
#pragma unroll
              for (int q = 0; q < 4; ++q) o[q] = __float_as_uint(v[c][4 * t + q]);
              so.store(off + 8 * c * ld4 + 16 * t, o);
            }
        } else {                                       // kRouterDx
          so.at(p.out0 + static_cast<long>(row0 + rs0) * p.ldo + n0, rows - rs0, ld2, skip2);
#pragma unroll
          for (int c = 0; c < 2; ++c) {
            const uint32_t off = off8(ld2) + 8 * c * ld2;
            float old[8];
            unpack8(so.load(off), old);
#pragma unroll
            for (int q = 0; q < 8; ++q) v[c][q] = p.accumulate ? v[c][q] + old[q] : v[c][q];
            so.store(off, pack8(v[c]));
          }
        }
      }
    }
    if (nxt.exists == 0) break;
    cur = nxt;
  }
  Loop::finish();
}

// ============================================================================================
// Weight-gradient kernels: out[e] (M x N) = lhs[rows of e, M]^T * rhs[rows of e, N]
// Output rows below `m_split` go to out0[e], the rest to out1[e] (gate / up share one launch).
//
// The reduction runs over the rows of an expert, so its length follows the routing.  Under skewed
// routing a few experts own most rows; to keep every workgroup's share bounded, the rows of an expert
// are cut into chunks of at most `chunk_rows`, one work item per (chunk, output tile).  An expert with a
// single chunk is written directly.  The chunks of a split expert leave fp32 partial tiles in the
// workspace, and a second kernel adds them in chunk order and rounds once -- the same result on every
// run, unlike atomic accumulation.  Items are ordered by descending expert size so the long ones start first.
// ============================================================================================
struct WgradItems {
  int32_t* count;        // [5]: number of items, of split experts and of experts without rows; the next piece of zeros of each product
  int32_t* expert;       // [max_items]; the experts without rows follow those of the items
  int32_t* k0;           // [max_items] first row of the chunk
  int32_t* k1;           // [max_items] one past its last row
  int32_t* slot;         // [max_items] partial-tile slot, or -1: write the result directly
  int32_t* split_expert; // [max_split]
  int32_t* split_slot0;  // [max_split]
  int32_t* split_n;      // [max_split]
  int max_items, max_split, max_slots;
};

__device__ __forceinline__ void build_wgrad_items(const int32_t* __restrict__ offsets, int E, int P, int chunk_rows, WgradItems it) {
  __shared__ int32_t cnt[kMaxExperts];      // rows per expert
  __shared__ int32_t order[kMaxExperts];    // expert at each rank (descending size, ties by index)
  __shared__ int32_t scan_items[kMaxExperts];
  __shared__ int32_t scan_slots[kMaxExperts];
  __shared__ int32_t scan_split[kMaxExperts];
  const int e = threadIdx.x;
  int begin = 0, c = -1;
  if (e < E) {
    begin = min(max(offsets[e], 0), P);
    c = min(max(offsets[e + 1], begin), P) - begin;
  }
  cnt[e] = c;
  __syncthreads();
  if (e < E) {
    int rank = 0;
    for (int o = 0; o < E; ++o) rank += (cnt[o] > c || (cnt[o] == c && o < e)) ? 1 : 0;
    order[rank] = e;
  }
  __syncthreads();
  // thread r now speaks for the expert of rank r
  int my_e = -1, my_n = 0, my_c = 0;
  if (e < E) {
    my_e = order[e];
    my_c = cnt[my_e];
    my_n = max(1, (my_c + chunk_rows - 1) / chunk_rows);
  }
  const int split = my_n > 1 ? 1 : 0;
  scan_items[e] = my_n;
  scan_slots[e] = split ? my_n : 0;
  scan_split[e] = split;
  __syncthreads();
  for (int o = 1; o < 1024; o <<= 1) {
    const int a = e >= o ? scan_items[e - o] : 0, b = e >= o ? scan_slots[e - o] : 0, d = e >= o ? scan_split[e - o] : 0;
    __syncthreads();
    scan_items[e] += a; scan_slots[e] += b; scan_split[e] += d;
    __syncthreads();
  }
  if (e < E) {
    const int first = scan_items[e] - my_n, slot0 = scan_slots[e] - (split ? my_n : 0), sidx = scan_split[e] - split;
    const int row0 = min(max(offsets[my_e], 0), P);
    // the host sizes the lists for the worst case; offsets that are not a monotone scan ending at P cannot overflow them
    const bool fits = slot0 + my_n <= it.max_slots && sidx < it.max_split;
    for (int j = 0; j < my_n && first + j < it.max_items; ++j) {
      it.expert[first + j] = my_e;
      it.k0[first + j] = row0 + (fits || !split ? j * chunk_rows : 0);
      it.k1[first + j] = fits || !split ? row0 + min(my_c, (j + 1) * chunk_rows) : (j == 0 ? row0 + my_c : row0);
      it.slot[first + j] = split && fits ? slot0 + j : (split && j > 0 ? -2 : -1);   // -2: nothing to do
    }
    if (split && fits) {
      it.split_expert[sidx] = my_e;
      it.split_slot0[sidx] = slot0;
      it.split_n[sidx] = my_n;
    }
  }
  // An expert without rows has no item: a tile of zeros would run two empty slabs and hold up the rings of a workgroup that
  // has rows to multiply.  They are the last ones of the order; workgroups store their zeros behind their last tile (pre-routed
  // steps of 32 experts, most of them empty: 144 rows, d = 512, f = 704 107 -> 100 us, 1500 rows, d = 1024, f = 1408 230 -> 214).
  if (e < E && my_c == 0 && (e == 0 || cnt[order[e - 1]] > 0)) {
    it.count[0] = min(scan_items[e] - 1, it.max_items);
    it.count[2] = min(E - e, it.max_items - it.count[0]);
  }
  if (e == E - 1 && my_c > 0) {
    it.count[0] = min(scan_items[e], it.max_items);
    it.count[2] = 0;
  }
  if (e == 1023) {
    it.count[1] = min(scan_split[1023], it.max_split);
    it.count[3] = it.count[4] = 0;
  }
}

// entries of padding behind the list of row tokens: a tile of 256 rows begins at most at the last row, and the weight gradients'
// scalar loads run one slab ahead and over at least two slabs, up to 3 * 64 entries past a chunk's first row or 2 * 64 past its last
constexpr int kRowTokenPad = 256;

// Everything a pass needs before its first product, in one launch: block 0 builds the (expert, row tile)
// list, block 1 the weight-gradient work items (backward only), the remaining blocks expand pair_of_row into
// the token (and combine weight) of every expert-ordered row (gathered passes only).
struct ScheduleArgs {
  const int32_t* offsets; int E, P;
  int bm; RowTiles rt;
  int chunk_rows; WgradItems items;      // chunk_rows == 0: no weight-gradient items
  const int32_t* pair_of_row;            // null: no row lists
  const float* topk_w; int T, k;
  int32_t* row_token; float* row_w;      // row_w may be null
};
__global__ __launch_bounds__(1024) void build_schedules_kernel(ScheduleArgs a) {
  if (blockIdx.x == 0) {
    build_row_tiles(a.offsets, a.E, a.P, a.bm, a.rt);
  } else if (blockIdx.x == 1) {
    if (a.chunk_rows > 0) build_wgrad_items(a.offsets, a.E, a.P, a.chunk_rows, a.items);
  } else {
    const int r = (blockIdx.x - 2) * 1024 + threadIdx.x;
    if (r >= a.P + kRowTokenPad) return;
    if (r >= a.P) { a.row_token[r] = 0; return; }
    const int pair = min(max(a.pair_of_row[r], 0), a.P - 1);
    a.row_token[r] = min(pair / a.k, a.T - 1);
    if (a.row_w) a.row_w[r] = a.topk_w[pair];
  }
}
static void launch_schedules(const ScheduleArgs& a, hipStream_t s) {
  const int blocks = 2 + (a.pair_of_row ? ceil_div(a.P + kRowTokenPad, 1024) : 0);
  MOE_LAUNCH("build_schedules", build_schedules_kernel, dim3(blocks), dim3(1024), 0, s, a);
}

struct WgradArgs {
  const bf16_t* lhs; long ld_lhs; int M;
  const bf16_t* rhs; long ld_rhs; int N;
  int E; int P;
  WgradItems items;
  int one_segment_items, chunk_rows;           // the router's (items is not used): chunks of chunk_rows rows, at least one
  int tiles_m, tiles_n;
  bf16_t* out0; bf16_t* out1; int m_split;     // out1 rows are (m - m_split)
  float* partial;                              // [max_slots][M][N]
  const int32_t* row_token;    // GATHER kernels: [P + padding], token of each expert-ordered row
  // a side job of the reduction launch of the gathered backward, taken from dW_down's arguments (null: none): the partial dot
  // products of the combine-weight gradient, one per (column slot, row), are added in slot order and scattered to [T, k]
  const float* dw_partial; int dw_slots; const int32_t* pair_of_row; float* dtopk_w;
};

// WHICH 0: dW_down, 1: [dW_gate; dW_up], 2: router (separate symbols so profiles tell them apart).
// GATHER: the operand that holds one row per token -- lhs for WHICH 0 (the output gradient), rhs for WHICH 1
// (the layer input) -- is the token-major matrix itself, and reduction row r reads its row row_token[r].
// THROUGH_L2: result stores that stay in the L2 until the kernel ends (see launch_wgrad).
template <int WHICH, class T, bool GATHER, bool THROUGH_L2>
__global__ __launch_bounds__(T::kThreads) __attribute__((amdgpu_waves_per_eu(T::kWavesPerSimd, T::kWavesPerSimd))) void wgrad_kernel(WgradArgs p) {
  static_assert(!GATHER || WHICH < 2, "the router's operands are token-major already");
  constexpr bool GA = GATHER && WHICH == 0, GB = GATHER && WHICH == 1;
  extern __shared__ __attribute__((aligned(16))) char lds[];
  constexpr int BM = T::BM, BN = T::BN, WM = T::WM, WN = T::WN, FN = T::FN;
  static_assert(FN == 4, "the epilogue takes the fragments of a row in two pairs");
  typedef MainLoop<T, true, true, GA, GB> Loop;
  constexpr bool ONE_SEGMENT = WHICH == 2;              // the router's: one segment of all rows, its chunks follow from their number
  const int n_items = ONE_SEGMENT ? p.one_segment_items : const_list(p.items.count)[0];
  // order of a work item's tiles: row tile fastest for [dW_gate; dW_up] (neighbouring workgroups share the rhs panel;
  // measured 6 % faster at 512 rows per expert), column tile fastest for the others
  constexpr bool MT_FASTEST = WHICH == 1;
  auto sc = [](int v) { return scalar(v); };
  const WgradWalk walk = wgrad_walk(n_items, MT_FASTEST ? p.tiles_n : p.tiles_m, p.tiles_m * p.tiles_n, static_cast<int>(gridDim.x), sc);
  // This workgroup's tiles, the next one located while one is multiplied
  struct At { int e, slot, begin, end, m0, n0, exists; };   // (`exists` is a number: see the row-grouped kernel)
  auto locate = [&](int& block) {
    At t{};
    for (;; block += gridDim.x) {
      const WgradTile at = wgrad_tile(walk, block, sc);
      t.exists = scalar(at.exists ? 1 : 0);
      if (!at.exists) return t;
      const int item = at.item, vi = at.tile;
      const int fast = MT_FASTEST ? p.tiles_m : p.tiles_n, slow_i = scalar(vi / fast), fast_i = vi - slow_i * fast;
      t.m0 = (MT_FASTEST ? fast_i : slow_i) * BM;
      t.n0 = (MT_FASTEST ? slow_i : fast_i) * BN;
      if constexpr (ONE_SEGMENT) {
        t.slot = n_items > 1 ? item : -1;
        t.begin = item * p.chunk_rows;
        t.end = min(p.P, t.begin + p.chunk_rows);
        return t;
      }
      t.slot = const_list(p.items.slot)[item];
      if (t.slot == -2) continue;
      t.e = const_list(p.items.expert)[item];
      t.begin = const_list(p.items.k0)[item];
      t.end = const_list(p.items.k1)[item];
      return t;
    }
  };
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  // The zeros of the experts without rows, 128 KiB at a time.  Workgroups without a tile store them while the others multiply, if
  // at least half of those launched have none; else whoever has no tile left takes the next piece, by a counter: a fixed share
  // for each leaves the workgroups of the longest experts theirs (1500 rows: the two products 83 us, by the counter 74).  With few
  // tiles the counter's round trip to memory is what a workgroup with a tile ends on (144 rows: 25 us, without it 22).
  auto store_zeros = [&] {
    if constexpr (!ONE_SEGMENT) {
      constexpr int kPer = 8, kPieces = kPer * T::kThreads;                   // 16-byte pieces
      int M = p.M, N = p.N;
      int32_t* count = p.items.count;
      asm volatile("" : "+s"(M), "+s"(N), "+s"(count));  // (nothing of this is worked out ahead of the tiles and kept)
      const long of_out0 = static_cast<long>(p.m_split) * N / 8, of_expert = static_cast<long>(M) * N / 8;
      const int per_e = static_cast<int>((of_expert + kPieces - 1) / kPieces), n = const_list(count)[2] * per_e;
      const int idle = max(walk.grid - walk.total, 0);
      const bool only_idle = 2 * idle >= walk.grid;
      int c = static_cast<int>(blockIdx.x) - walk.total, next = 0;
      if (n == 0 || (only_idle && c < 0)) return;
      const int tid = wave * 64 + lane_id();
      int32_t* const word = reinterpret_cast<int32_t*>(lds);
      __syncthreads();                                  // (the rings are done with)
      while (c < n) {
        if (!only_idle && tid == 0) next = idle + atomicAdd(count + 3 + WHICH, 1);
        if (c >= 0) {
          const int j = scalar(c / per_e);
          const long e = const_list(p.items.expert)[n_items + j], first = static_cast<long>(c - j * per_e) * kPieces;
#pragma unroll
          for (int q = 0; q < kPer; ++q) {
            const long i = first + q * T::kThreads + tid;
            if (i < of_expert) store16(i < of_out0 ? p.out0 + (e * of_out0 + i) * 8 : p.out1 + (e * (of_expert - of_out0) + i - of_out0) * 8, u32x4{0, 0, 0, 0});
          }
        }
        c += idle;
        if (!only_idle) {
          if (tid == 0) *word = next;
          __syncthreads();
          c = scalar(*word);
          __syncthreads();
        }
      }
    }
  };
  int block = blockIdx.x;
  At cur = locate(block);
  if (cur.exists == 0) {
    store_zeros();
    return;
  }

  const int lane = threadIdx.x & 63;
  const int wm = wave / T::WGN, wn = wave % T::WGN;
  const int a_row = wm * WM, b_row = wn * WN;
  Loop ml;
  auto load = [&](const At& t) {
    Operand opA, opB;
    const int mrows = scalar(min(BM, p.M - t.m0)), ncols = scalar(min(BN, p.N - t.n0));
    opA.ld = p.ld_lhs;
    opA.half[0] = p.lhs + (GA ? 0L : static_cast<long>(t.begin) * p.ld_lhs) + t.m0;
    opA.half[1] = opA.half[0] + BM / 2;
    opA.valid[0] = min(mrows, BM / 2);
    opA.valid[1] = max(mrows - BM / 2, 0);
    opA.gather = GA ? p.row_token : nullptr;
    opA.grow = t.begin;
    opB.ld = p.ld_rhs;
    opB.gather = GB ? p.row_token : nullptr;
    opB.grow = t.begin;
    opB.half[0] = p.rhs + (GB ? 0L : static_cast<long>(t.begin) * p.ld_rhs) + t.n0;
    opB.half[1] = opB.half[0] + BN / 2;
    opB.valid[0] = min(ncols, BN / 2);
    opB.valid[1] = max(ncols - BN / 2, 0);
    ml.load_tile(opA, opB, nullptr, t.end - t.begin);
  };
  ml.prepare(lds);
  load(cur);
  ml.fill();

  for (;;) {
    block += gridDim.x;
    const At nxt = locate(block);
    Acc<T> acc;
    zero_acc<T>(acc);
    ml.template tile<true>(Loop::slabs_run(cur.end - cur.begin), a_row, b_row, true, acc, [&] { load(nxt); });

    const int el = not_before_here(lane);              // this lane, for the epilogue
    const uint32_t scratch = ml.scratch();
    static_assert(Loop::kScratch >= 2048, "strips of 16 rows");
    const int mrows = scalar(min(BM, p.M - cur.m0)), ncols = scalar(min(BN, p.N - cur.n0));
    const uint32_t skip = static_cast<uint32_t>(cur.n0);
    const int l3 = el >> 3, l7 = el & 7;
    if (cur.slot >= 0) {                               // chunk of a split expert: fp32 partial tile, 16 rows x 32 columns at a time
      const uint32_t ld4 = static_cast<uint32_t>(p.N) * 4u;
      const uint32_t at_w = scratch + (el & 15) * 128 + (((el >> 4) ^ (el & 7)) << 4), at_r = scratch + l3 * 128 + ((l7 ^ l3) << 4);
      StripRows so;
      so.at<WM>(p.partial + (static_cast<long>(cur.slot) * p.M + cur.m0 + a_row) * p.N + cur.n0, mrows - a_row, ld4, skip * 4u);
#pragma unroll
      for (int i = 0; i < T::FM; ++i)
#pragma unroll
        for (int q = 0; q < 2; ++q) {
          lds_park16(at_w, __builtin_bit_cast(u32x4, acc[i][2 * q]));
          lds_park16(at_w ^ 64, __builtin_bit_cast(u32x4, acc[i][2 * q + 1]));
          u32x4 v[2];
          lds_fetch(at_r, at_r + 1024, v[0], v[1]);
          const int c = b_row + 32 * q + 4 * l7;
#pragma unroll
          for (int h = 0; h < 2; ++h) so.store(off_if(c < ncols, (16 * i + 8 * h + l3) * ld4 + c * 4u, kOffNone), v[h]);
        }
    } else {                                           // whole expert: rounded once
      const uint32_t ld2 = static_cast<uint32_t>(p.N) * 2u;
      const StripBf16 strip(scratch, el);
      const int c = b_row + 8 * l7;
      // the tile's rows below m_split belong to out0, the others to out1
      const int below = min(max(p.m_split - cur.m0, 0), mrows);
#pragma nounroll
      for (int half = 0; half < 2; ++half) {
        const int lo = half == 0 ? 0 : below, hi = half == 0 ? below : mrows;
        if (lo >= hi) continue;
        const int first = max(lo, a_row);                // of this wave's rows
        bf16_t* out = half == 0 ? p.out0 + (static_cast<long>(cur.e) * p.m_split + cur.m0 + first) * p.N
                                : p.out1 + (static_cast<long>(cur.e) * (p.M - p.m_split) + (cur.m0 + first - p.m_split)) * p.N;
        StripRows so;
        so.at<WM>(out + cur.n0, min(hi, a_row + WM) - first, ld2, skip * 2u);
#pragma unroll
        for (int i = 0; i < T::FM; ++i) {
#pragma unroll
          for (int j = 0; j < FN; ++j) strip.park(j, acc[i][j]);
          u32x4 v[2];
          strip.fetch(v[0], v[1]);
#pragma unroll
          for (int h = 0; h < 2; ++h) {
            const int r = a_row + 16 * i + 8 * h + l3 - first;
            so.store_as<THROUGH_L2>(off_if(c < ncols && r >= 0, r * ld2 + c * 2u, kOffNone), v[h]);
          }
        }
      }
    }
    if (nxt.exists == 0) break;
    cur = nxt;
  }
  Loop::finish();
  store_zeros();
}

// out[e] = bf16( sum over the chunks of a split expert, in chunk order, of its fp32 partial tiles ), for one weight gradient
// or for both of the experts' (which share their work items) in one launch
// (with balanced routing there are no split experts, and the launch is blocks that read one counter and leave)
struct WgradReduceArgs { WgradArgs a, b; };            // b.partial == null: a alone
// AT_ONCE: partial tiles requested together.  Few chunks (the experts'): 4; 8 is 6 % slower at 151 MB of partial tiles.  Many (the
// router's, 32 and 64): 8, 16.3 -> 13.6 and 24.6 -> 20.4 us.
template <int AT_ONCE>
__global__ __launch_bounds__(256) void wgrad_reduce_kernel(WgradReduceArgs args) {
  const WgradArgs& p = args.a;
  if (p.dw_partial) {                                  // dtopk_w[pair_of_row[r]] = sum over the column slots, in slot order
    for (int r = blockIdx.x * 256 + threadIdx.x; r < p.P; r += gridDim.x * 256) {
      // 16 slots requested together (one after the other, 32 slots of 8192 rows took 18 us), added in order
      float s = 0.0f;
      for (int j = 0; j < p.dw_slots; j += 16) {
        float v[16];
#pragma unroll
        for (int u = 0; u < 16; ++u) v[u] = p.dw_partial[static_cast<long>(min(j + u, p.dw_slots - 1)) * p.P + r];
#pragma unroll
        for (int u = 0; u < 16; ++u) s = j + u < p.dw_slots ? s + v[u] : s;
      }
      p.dtopk_w[min(max(p.pair_of_row[r], 0), p.P - 1)] = s;
    }
  }
  // every (split expert, 8 outputs) pair is one unit of a single grid-strided loop: the launch is latency-bound (a unit is
  // one round of loads and one store), so the split experts are reduced side by side, not one after the other
  const int n_split = p.one_segment_items ? (p.one_segment_items > 1 ? 1 : 0) : p.items.count[1];
  const long per_a = static_cast<long>(p.M) * p.N / 8;                 // N is a multiple of 8: a unit lies in one row
  const long per = per_a + (args.b.partial ? static_cast<long>(args.b.M) * args.b.N / 8 : 0L);
  for (long unit = static_cast<long>(blockIdx.x) * 256 + threadIdx.x; unit < n_split * per; unit += static_cast<long>(gridDim.x) * 256) {
    const int s = static_cast<int>(unit / per);
    const long u = unit - s * per;
    const WgradArgs& q = u < per_a ? args.a : args.b;
    const long i = (u < per_a ? u : u - per_a) * 8, mn = static_cast<long>(q.M) * q.N;
    const int e = p.one_segment_items ? 0 : p.items.split_expert[s], n = p.one_segment_items ? p.one_segment_items : p.items.split_n[s];
    const float* part = q.partial + (p.one_segment_items ? 0L : static_cast<long>(p.items.split_slot0[s])) * mn;
    float acc[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    for (int j = 0; j < n; j += AT_ONCE) {                 // requested together, added in slot order
      float v[AT_ONCE][8];
#pragma unroll
      for (int t = 0; t < AT_ONCE; ++t) read8(part + min(j + t, n - 1) * mn + i, v[t]);   // past the last slot: re-read it, not added
#pragma unroll
      for (int t = 0; t < AT_ONCE; ++t) {
        if (j + t < n) {
#pragma unroll
          for (int c = 0; c < 8; ++c) acc[c] += v[t][c];
        }
      }
    }
    const int m = static_cast<int>(i / q.N), col = static_cast<int>(i % q.N);
    bf16_t* out = m < q.m_split ? q.out0 + (static_cast<long>(e) * q.m_split + m) * q.N
                                : q.out1 + (static_cast<long>(e) * (q.M - q.m_split) + (m - q.m_split)) * q.N;
    store16(out + col, pack8(acc));
  }
}

// ============================================================================================
// Host side
// ============================================================================================
// Tile shapes in use.
//   TileBig: 256 x 256 outputs, 64-wide slabs, one 8-wave workgroup per CU (2 x 4 wavefronts of 128 x 64), rings of
//     2 + 3 slab buffers of 32 KiB.  A slab row is a whole 128-byte line: the fewest L2 requests per flop that fit the CU.
//   TileBigW16: the same tile and rings under 16 waves (4 x 4 of 64 x 64, four per SIMD, 128 VGPRs) for the weight
//     gradients: both their operands are read transposed (twice the LDS instructions per fragment), and four
//     waves per SIMD cover that better: [dW_gate; dW_up] 510-516 us against 529-532 with 8 waves at 512 rows per expert,
//     1837 against 1940 at 2560; dW_down 259 against 261 and 911 against 967.  The row products keep 8 waves.
//   TileRouter: 64 x 128 x 64 for the skinny products with N = E, two workgroups per CU.
typedef Tile<256, 256, 64, 2, 4, 2, 3> TileBig;
typedef Tile<256, 256, 64, 4, 4, 2, 3> TileBigW16;
typedef Tile<64, 128, 64, 2, 2, 2, 3> TileRouter;

// Row-grouped products of experts with few rows: a quarter of the tile, two workgroups of four waves per CU.  These products
// stream the weights once; what they lack with the large tile is workgroups (a row tile per expert) and something to run
// while a workgroup starts or ends.  The same sums in the same order: results are bit-identical.
typedef Tile<128, 128, 64, 2, 2, 2, 3> TileFew;
// Rows of a pass's row tiles.  Measured, forward / forward and backward, large tile -> small:
//   E = 16, d = 1024, f = 2048 (64 large tiles onto d): 2 rows per expert 65 -> 59 us / 207 -> 183, 64 rows 75 -> 69 / 239 -> 221,
//     125 rows 88 -> 82 / 282 -> 259;  E = 8, d = 4096, f = 3072 (128): 2 rows 155 -> 134 / 473 -> 413, 64 rows 175 -> 159 / 540 -> 504;
//   E = 60, d = 1024, f = 1408 (240): 4 rows 125 -> 121 / 369 -> 366, 93 rows 145 -> 144 / 461 -> 459;
//   E = 128, d = 2048, f = 768 (1024, four rounds of the 256 CUs): 4 rows 244 -> 237, 64 rows 275 -> 273, 96 rows 285 -> 287, 128 rows
//     305 -> 356 (half of the experts need a second tile, which reads their weights again); with the backward 856 -> 875 at 64 rows
//     and 926 -> 959 at 96 (its weights are read across the reduction, 256 bytes at a time instead of 512).
// So: on average at most 128 rows per expert where the large tiles onto d leave CUs without work, and 64 in a forward pass of any size.
// The average stands for uneven routing too (Zipf with exponent 1.2; half of the rows on one expert): E = 16, d = 1024, f = 2048, 125 rows
// 120 -> 93 us / 315 -> 258 and 106 -> 90 / 312 -> 265; E = 63, d = 1024, f = 3072, 128 rows 475 -> 413 / 1547 -> 1449 and 428 -> 362 / 1471 ->
// 1307; E = 128, d = 2048, f = 768, 64 rows 358 -> 317 and 339 -> 292 forward.  It loses where wide experts spill into a second round of
// workgroups (E = 8, d = 4096, f = 3072, 128 rows: 190 -> 224 / 651 -> 682, 191 -> 209 / 632 -> 638; at 64 rows 188 -> 169 / 602 -> 558) and in the
// forward of large calls with every row on one expert (E = 63 above 204 -> 235 / 952 -> 943; E = 512, d = 2048, f = 768, 64 rows 325 -> 386).
static int row_bm(int P, int E, int d, bool backward) {
  const bool idle = static_cast<long>(E) * ceil_div(d, TileBig::BN) < 256 && P <= 128L * E;
  return idle || (!backward && P <= 64L * E) ? TileFew::BM : TileBig::BM;
}
// bound used for workspace sizing: the smallest row tile gives the longest list
static int max_row_tiles(int P, int E) { return ceil_div(P, 128) + E; }

// Rows per reduction chunk of the weight gradients: long enough that the fp32 partial tiles stay a small
// part of the traffic, short enough that the largest work item is a small part of the launch.  At most
// 2 * ceil(P / chunk) <= 64 partial slots can ever be needed (an expert is split only if it has more than
// one chunk, and the chunks of split experts hold more than half their rows each but the last).  The floor of
// 2048 rows is the measured optimum when 16 experts share 16K rows with two thirds of them on one expert
// (1024: a third more partial traffic; 3072: too few work items per XCD).
static int wgrad_chunk_rows(int P) { return std::max(2048, static_cast<int>(align_up(static_cast<size_t>(ceil_div(P, 32)), 256))); }
static int wgrad_max_items(int P, int E) { return E + ceil_div(P, wgrad_chunk_rows(P)); }
static int wgrad_max_split(int P, int E) { return std::max(1, std::min(E, ceil_div(P, wgrad_chunk_rows(P)))); }
static int wgrad_max_slots(int P) { return 2 * ceil_div(P, wgrad_chunk_rows(P)); }
// The router's weight gradient has a single "expert" of all T rows and only E x d outputs: shorter chunks
// (at least 64 of them) so that the launch fills the chip.
static int router_chunk_rows(int T) { return std::max(256, static_cast<int>(align_up(static_cast<size_t>(ceil_div(T, 64)), 256))); }

struct WsLayout {
  size_t tiles_count, tiles_entry, dgu, g, u, items, partial, total;
};
static WsLayout ws_layout(int P, int d, int f, int E, bool need_dgu, bool need_gu) {
  WsLayout w{};
  size_t off = 0;
  w.tiles_count = off; off += 256;
  w.tiles_entry = off; off += align_up(static_cast<size_t>(max_row_tiles(P, E)) * sizeof(TileEntry), 256);
  const size_t pf = align_up(static_cast<size_t>(P) * f * 2, 256);
  w.dgu = off; if (need_dgu) off += 2 * pf;
  w.g = off; if (need_gu) off += pf;
  w.u = off; if (need_gu) off += pf;
  w.items = off; w.partial = off;
  if (need_dgu) {                                      // backward only: weight-gradient schedule and partial tiles
    const size_t it = align_up(static_cast<size_t>(wgrad_max_items(P, E)) * sizeof(int32_t), 256);
    const size_t sp = align_up(static_cast<size_t>(wgrad_max_split(P, E)) * sizeof(int32_t), 256);
    off += 256 + 4 * it + 3 * sp;
    w.partial = off;
    // dW_down's, then [dW_gate; dW_up]'s: one reduction launch for both, 5 us less of each step, for a third of this memory (64 slots,
    // d = 2048, f = 768: 1208 MB, with two launches 805)
    off += align_up(static_cast<size_t>(wgrad_max_slots(P)) * 3 * f * d * sizeof(float), 256);
  }
  w.total = off + 256;
  return w;
}

size_t ffn_fwd_ws_bytes_bf16(int P, int d, int f, int E) { return ws_layout(P, d, f, E, false, false).total; }
size_t ffn_bwd_ws_bytes_bf16(int P, int d, int f, int E, int have_saved) {
  return ws_layout(P, d, f, E, true, !have_saved).total;
}

static RowTiles row_tiles_at(void* ws, const WsLayout& w, int P, int E, int bm) {
  char* b = static_cast<char*>(ws);
  RowTiles rt;
  rt.max_tiles = max_row_tiles(P, E);
  rt.bm = bm;
  rt.count = reinterpret_cast<int32_t*>(b + w.tiles_count);
  rt.entry = reinterpret_cast<TileEntry*>(b + w.tiles_entry);
  return rt;
}

static WgradItems wgrad_items_at(void* ws, const WsLayout& w, int P, int E) {
  char* b = static_cast<char*>(ws) + w.items;
  WgradItems it;
  it.max_items = wgrad_max_items(P, E);
  it.max_split = wgrad_max_split(P, E);
  it.max_slots = wgrad_max_slots(P);
  const size_t li = align_up(static_cast<size_t>(it.max_items) * sizeof(int32_t), 256);
  const size_t ls = align_up(static_cast<size_t>(it.max_split) * sizeof(int32_t), 256);
  it.count = reinterpret_cast<int32_t*>(b); b += 256;
  it.expert = reinterpret_cast<int32_t*>(b); b += li;
  it.k0 = reinterpret_cast<int32_t*>(b); b += li;
  it.k1 = reinterpret_cast<int32_t*>(b); b += li;
  it.slot = reinterpret_cast<int32_t*>(b); b += li;
  it.split_expert = reinterpret_cast<int32_t*>(b); b += ls;
  it.split_slot0 = reinterpret_cast<int32_t*>(b); b += ls;
  it.split_n = reinterpret_cast<int32_t*>(b);
  return it;
}

// A kernel that needs more than 64 KiB of dynamic LDS has to be granted it once per device.  Each kernel has its
// own set of flags (a static of its launcher's template instance); the status is kept, and a failure is reported
// through the call's launch status instead of surfacing later as an opaque launch error.
constexpr int kMaxDevices = 64;
struct LdsGrant { std::once_flag once[kMaxDevices]; hipError_t status[kMaxDevices] = {}; };
static bool allow_lds(LdsGrant& g, const void* kernel, int bytes, const char* name) {
  int dev = 0;
  hipError_t err = hipGetDevice(&dev);
  if (err == hipSuccess && (dev < 0 || dev >= kMaxDevices)) err = hipErrorInvalidDevice;
  if (err == hipSuccess) {
    std::call_once(g.once[dev], [&] { g.status[dev] = hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize, bytes); });
    err = g.status[dev];
  }
  if (err != hipSuccess) note_hip_failure(name, err);
  return err == hipSuccess;
}

// The products' workgroups stay on their CU and take tile after tile: as many as run at once, or fewer if there are fewer tiles.
constexpr int kCus = 256;
static unsigned padded_grid(int tiles) { return static_cast<unsigned>(ceil_div(tiles < 1 ? 1 : tiles, kXcds) * kXcds); }

static unsigned resident_grid(int tiles, int blocks_per_cu) { return std::min(padded_grid(tiles), static_cast<unsigned>(kCus * blocks_per_cu)); }

template <int KIND, class T, bool FUSED = false, bool OPTION = false>
static void launch_row_t(RowArgs p, int P, int E, hipStream_t s) {
  static const char* const names[6] = {"ffn_gate_up", "ffn_down", "ffn_dact", "ffn_dx", "router_logits", "router_dx"};
  static LdsGrant grant;
  if (!allow_lds(grant, reinterpret_cast<const void*>(&row_grouped_kernel<KIND, T, FUSED, OPTION>), T::kLdsBytes, names[KIND])) return;
  p.n_tiles_n = ceil_div(p.N, KIND == kGateUp ? T::BN / 2 : T::BN);
  const unsigned grid = resident_grid((ceil_div(P, T::BM) + E) * p.n_tiles_n, T::kBlocksPerCu);
  MOE_LAUNCH(names[KIND], (row_grouped_kernel<KIND, T, FUSED, OPTION>), dim3(grid), dim3(T::kThreads), T::kLdsBytes, s, p);
}

template <int KIND, bool FUSED = false, bool OPTION = false>
static void launch_row(const RowArgs& p, int P, int E, hipStream_t s) {
  if (p.rt.bm == TileFew::BM) launch_row_t<KIND, TileFew, FUSED, OPTION>(p, P, E, s);
  else launch_row_t<KIND, TileBig, FUSED, OPTION>(p, P, E, s);
}

template <int WHICH, bool GATHER, bool THROUGH_L2>
static void launch_wgrad_as(WgradArgs p, hipStream_t s) {
  typedef TileBigW16 T;
  static LdsGrant grant;
  if (!allow_lds(grant, reinterpret_cast<const void*>(&wgrad_kernel<WHICH, T, GATHER, THROUGH_L2>), T::kLdsBytes, "wgrad")) return;
  p.tiles_m = ceil_div(p.M, T::BM);
  p.tiles_n = ceil_div(p.N, T::BN);
  // units are dealt to the XCDs in groups of 8, the last group may be partial: up to 8 more units than items
  const int max_items = WHICH == 2 ? p.one_segment_items : p.items.max_items;
  const unsigned grid = resident_grid(p.tiles_m * p.tiles_n * (max_items + kXcds), T::kBlocksPerCu);
  MOE_LAUNCH(WHICH == 0 ? "wgrad_down" : WHICH == 1 ? "wgrad_gate_up" : "wgrad_router", (wgrad_kernel<WHICH, T, GATHER, THROUGH_L2>), dim3(grid),
             dim3(T::kThreads), T::kLdsBytes, s, p);
}
// Result rows that are no whole number of lines go through the L2, where the pieces of a line meet: past it they reach memory one
// by one, and the next tile waits for their acknowledgements (E = 128, 45 rows, d = 568, f = 1216: gate/up 209 -> 101 us, step 593
// -> 530).  Whole lines go past it: through it 8 rows of d = 2048, f = 768 take 156 instead of 145 us, the step 774 instead of 701.
template <int WHICH, bool GATHER = false>
static void launch_wgrad(const WgradArgs& p, hipStream_t s) {
  if (p.N * 2 % 128 != 0) launch_wgrad_as<WHICH, GATHER, true>(p, s);
  else launch_wgrad_as<WHICH, GATHER, false>(p, s);
}
// the partial tiles of one weight gradient, or (b given) of both of the experts' in one launch behind the two products
static void launch_wgrad_reduce(const char* name, const WgradArgs& a, const WgradArgs* b, hipStream_t s) {
  WgradReduceArgs r{a, {}};
  if (b) r.b = *b;
  // the reduction loops are grid-strided: a launch with nothing to reduce (balanced routing) should cost as little as a launch can
  // (room for two split experts per pass of the loop; more only repeat it)
  const long outputs = static_cast<long>(a.M) * a.N + (b ? static_cast<long>(b->M) * b->N : 0L);
  const long blocks = std::max(2 * ((outputs + 2047) / 2048), a.dw_partial ? (static_cast<long>(a.P) + 255) / 256 : 1L);
  const dim3 grid(static_cast<unsigned>(std::min(blocks, 2048L)));
  if (a.one_segment_items) MOE_LAUNCH(name, wgrad_reduce_kernel<8>, grid, dim3(256), 0, s, r);
  else MOE_LAUNCH(name, wgrad_reduce_kernel<4>, grid, dim3(256), 0, s, r);
}

// row_token == null: xp is in expert order; else xp is the token-major input and rows are gathered from it
static void launch_gate_up(const void* xp, const void* wg, const void* wu, int P, int d, int f, int E,
                           const RowTiles& rt, void* G, void* U, void* act, hipStream_t s,
                           const int32_t* row_token = nullptr, const float* row_w = nullptr) {
  RowArgs p{};
  p.row_token = row_token;
  p.row_w = row_w;
  p.a = static_cast<const bf16_t*>(xp); p.lda = d;
  p.w0 = static_cast<const bf16_t*>(wg); p.w1 = static_cast<const bf16_t*>(wu);
  p.w_expert_stride = static_cast<long>(f) * d; p.ldw = d;
  p.K = d; p.N = f; p.P = P; p.rt = rt;
  p.out0 = static_cast<bf16_t*>(G); p.out1 = static_cast<bf16_t*>(U); p.out2 = static_cast<bf16_t*>(act); p.ldo = f;
  // A wave's G, U and activation fill half a line per row.  Written around the L2 (non-temporal), both halves go to memory on
  // their own; written through it, another wave's half joins them, but they displace weights and are still being written back
  // when the next launch starts.  Joining them pays where all three are written by experts with many rows -- 40960 tokens,
  // d = 2048, E = 128, k = 8, f = 768: 1760 -> 1681 us, 8192 tokens 424 -> 411 (step 2092 -> 2082), 16384 rows on 16 experts
  // 106 -> 102 (594 -> 589) -- and costs with few rows (1531 tokens, 96 rows per expert: gate/up 155 -> 161, down 89 -> 96) or
  // with the activation alone (8192 tokens forward: 709 -> 709; 2047 tokens: 313 -> 317).  256 rows per expert: step 1349 and 1350.
  const bool through_l2 = G && act && P >= 256L * E;
  if (through_l2) {
    if (row_token) launch_row_t<kGateUp, TileBig, true, true>(p, P, E, s);
    else launch_row_t<kGateUp, TileBig, false, true>(p, P, E, s);
  } else if (row_token) {
    launch_row<kGateUp, true>(p, P, E, s);
  } else {
    launch_row<kGateUp>(p, P, E, s);
  }
}

static void launch_down(const void* act, const void* wd, int P, int d, int f, int E,
                        const RowTiles& rt, void* yp, hipStream_t s) {
  RowArgs p{};
  p.a = static_cast<const bf16_t*>(act); p.lda = f;
  p.w0 = static_cast<const bf16_t*>(wd); p.w_expert_stride = static_cast<long>(d) * f; p.ldw = f;
  p.K = f; p.N = d; p.P = P; p.rt = rt;
  p.out0 = static_cast<bf16_t*>(yp); p.ldo = d;
  launch_row<kDown>(p, P, E, s);
}

static void launch_dx(const bf16_t* dgu, const void* wg, const void* wu, int P, int d, int f, int E,
                      const RowTiles& rt, void* dxp, hipStream_t s) {
  RowArgs p{};
  p.a = dgu; p.lda = 2L * f;
  p.w0 = static_cast<const bf16_t*>(wg); p.w1 = static_cast<const bf16_t*>(wu);
  p.w_expert_stride = static_cast<long>(f) * d; p.ldw = d;
  p.K = f; p.N = d; p.P = P; p.rt = rt;
  p.out0 = static_cast<bf16_t*>(dxp); p.ldo = d;
  launch_row<kDX>(p, P, E, s);
}

void ffn_fwd_bf16(const FfnFwdArgs& a) {
  const WsLayout w = ws_layout(a.P, a.d, a.f, a.E, false, false);
  const RowTiles rt = row_tiles_at(a.ws, w, a.P, a.E, row_bm(a.P, a.E, a.d, false));
  MOE_LAUNCH("build_row_tiles", build_row_tiles_kernel, dim3(1), dim3(1024), 0, a.stream, a.offsets, a.E, a.P, rt.bm, rt);
  launch_gate_up(a.xp, a.w_gate, a.w_up, a.P, a.d, a.f, a.E, rt, a.g_save, a.u_save, a.act, a.stream);
  launch_down(a.act, a.w_down, a.P, a.d, a.f, a.E, rt, a.yp, a.stream);
}

void ffn_bwd_bf16(const FfnBwdArgs& a) {
  const bool recompute = a.g_save == nullptr;
  const WsLayout w = ws_layout(a.P, a.d, a.f, a.E, true, recompute);
  const RowTiles rt = row_tiles_at(a.ws, w, a.P, a.E, row_bm(a.P, a.E, a.d, true));
  char* base = static_cast<char*>(a.ws);
  bf16_t* dgu = reinterpret_cast<bf16_t*>(base + w.dgu);       // [P, 2f] = [dG | dU]
  const bf16_t* G = static_cast<const bf16_t*>(a.g_save);
  const bf16_t* U = static_cast<const bf16_t*>(a.u_save);
  const WgradItems items = wgrad_items_at(a.ws, w, a.P, a.E);
  {
    ScheduleArgs sa{};
    sa.offsets = a.offsets; sa.E = a.E; sa.P = a.P; sa.bm = rt.bm; sa.rt = rt;
    sa.chunk_rows = wgrad_chunk_rows(a.P); sa.items = items;
    launch_schedules(sa, a.stream);
  }
  if (recompute) {
    bf16_t* Gr = reinterpret_cast<bf16_t*>(base + w.g);
    bf16_t* Ur = reinterpret_cast<bf16_t*>(base + w.u);
    launch_gate_up(a.xp, a.w_gate, a.w_up, a.P, a.d, a.f, a.E, rt, Gr, Ur, nullptr, a.stream);
    G = Gr; U = Ur;
  }
  {  // dA = dyp Wd, fused with the SwiGLU derivative -> [dG | dU]
    RowArgs p{};
    p.a = static_cast<const bf16_t*>(a.dyp); p.lda = a.d;
    p.w0 = static_cast<const bf16_t*>(a.w_down); p.w_expert_stride = static_cast<long>(a.d) * a.f; p.ldw = a.f;
    p.K = a.d; p.N = a.f; p.P = a.P; p.rt = rt;
    p.out0 = dgu; p.ldo = 2L * a.f; p.g = G; p.u = U;
    launch_row<kDAct>(p, a.P, a.E, a.stream);
  }
  launch_dx(dgu, a.w_gate, a.w_up, a.P, a.d, a.f, a.E, rt, a.dxp, a.stream);   // dxp = dG Wg + dU Wu
  float* partial = reinterpret_cast<float*>(base + w.partial);
  WgradArgs down{}, gate_up{};
  {  // dWd[e] = dyp^T act
    WgradArgs& p = down;
    p.lhs = static_cast<const bf16_t*>(a.dyp); p.ld_lhs = a.d; p.M = a.d;
    p.rhs = static_cast<const bf16_t*>(a.act); p.ld_rhs = a.f; p.N = a.f;
    p.E = a.E; p.P = a.P; p.items = items; p.partial = partial;
    p.out0 = static_cast<bf16_t*>(a.dw_down); p.out1 = p.out0; p.m_split = a.d;
    launch_wgrad<0>(p, a.stream);
  }
  {  // [dWg[e]; dWu[e]] = [dG | dU]^T xp
    WgradArgs& p = gate_up;
    p.lhs = dgu; p.ld_lhs = 2L * a.f; p.M = 2 * a.f;
    p.rhs = static_cast<const bf16_t*>(a.xp); p.ld_rhs = a.d; p.N = a.d;
    p.E = a.E; p.P = a.P; p.items = items; p.partial = partial + static_cast<size_t>(items.max_slots) * a.f * a.d;
    p.out0 = static_cast<bf16_t*>(a.dw_gate); p.out1 = static_cast<bf16_t*>(a.dw_up); p.m_split = a.f;
    launch_wgrad<1>(p, a.stream);
  }
  launch_wgrad_reduce("wgrad_reduce", down, &gate_up, a.stream);
}

// ============================================================================================
// The same two passes without the expert-ordered copies of the layer input and of the output gradient
// (the dispatch / return of Sec. 3.2.3 folded into the products that consume the rows):
//   forward   G, U, act, yp as above, rows read as x[token(r)]                              (no xp)
//   backward  dA = w_r dy[token(r)] Wd,  dWd = dy[token]^T (w act),  d w = <dy[token] Wd, act>,
//             [dWg; dWu] = [dG | dU]^T x[token]                                             (no dyp, no yp)
// token(r) = pair_of_row[r] / k and w_r = topk_w[pair_of_row[r]] are expanded once per call into two
// row-indexed lists; the list of tokens is padded so that the scalar loads that run one slab ahead of the
// weight-gradient products never leave it.
// ============================================================================================

// column slots of the combine-weight gradient's partial dot products: one per (column tile, wavefront column) of the dA product;
// dw_slots_max sizes the workspace
static int dw_slots_max(int f) { return ceil_div(f, TileBig::BN) * TileBig::WGN; }
static int dw_slots(const RowTiles& rt, int f) { return rt.bm == TileFew::BM ? ceil_div(f, TileFew::BN) * TileFew::WGN : dw_slots_max(f); }

struct GatherWs { size_t row_token, row_w, act_w, dw_partial, total; };
static GatherWs gather_ws(const WsLayout& w, int P, int f, bool bwd) {
  GatherWs g{};
  size_t off = w.total;
  g.row_token = off; off += align_up(static_cast<size_t>(P + kRowTokenPad) * sizeof(int32_t), 256);
  g.row_w = off; off += align_up(static_cast<size_t>(P) * sizeof(float), 256);
  g.act_w = off; g.dw_partial = off;
  if (bwd) {
    g.act_w = off; off += align_up(static_cast<size_t>(P) * f * 2, 256);
    g.dw_partial = off; off += align_up(static_cast<size_t>(dw_slots_max(f)) * P * sizeof(float), 256);
  }
  g.total = off;
  return g;
}
size_t ffn_fwd_gather_ws_bytes_bf16(int P, int d, int f, int E) {
  return gather_ws(ws_layout(P, d, f, E, false, false), P, f, false).total;
}
size_t ffn_bwd_gather_ws_bytes_bf16(int P, int d, int f, int E, int have_saved) {
  return gather_ws(ws_layout(P, d, f, E, true, !have_saved), P, f, true).total;
}

void ffn_fwd_gather_bf16(const FfnFwdGatherArgs& a) {
  const WsLayout w = ws_layout(a.P, a.d, a.f, a.E, false, false);
  const GatherWs g = gather_ws(w, a.P, a.f, false);
  const RowTiles rt = row_tiles_at(a.ws, w, a.P, a.E, row_bm(a.P, a.E, a.d, false));
  int32_t* row_token = reinterpret_cast<int32_t*>(static_cast<char*>(a.ws) + g.row_token);
  float* row_w = reinterpret_cast<float*>(static_cast<char*>(a.ws) + g.row_w);
  {
    ScheduleArgs sa{};
    sa.offsets = a.offsets; sa.E = a.E; sa.P = a.P; sa.bm = rt.bm; sa.rt = rt;
    sa.pair_of_row = a.pair_of_row; sa.T = a.T; sa.k = a.k; sa.row_token = row_token;
    if (a.topk_w) { sa.topk_w = a.topk_w; sa.row_w = row_w; }
    launch_schedules(sa, a.stream);
  }
  launch_gate_up(a.x, a.w_gate, a.w_up, a.P, a.d, a.f, a.E, rt, a.g_save, a.u_save, a.act, a.stream, row_token,
                 a.topk_w ? row_w : nullptr);
  launch_down(a.act, a.w_down, a.P, a.d, a.f, a.E, rt, a.yp, a.stream);
}

void ffn_bwd_gather_bf16(const FfnBwdGatherArgs& a) {
  const bool recompute = a.g_save == nullptr;
  const WsLayout w = ws_layout(a.P, a.d, a.f, a.E, true, recompute);
  const GatherWs gw = gather_ws(w, a.P, a.f, true);
  const RowTiles rt = row_tiles_at(a.ws, w, a.P, a.E, row_bm(a.P, a.E, a.d, true));
  char* base = static_cast<char*>(a.ws);
  bf16_t* dgu = reinterpret_cast<bf16_t*>(base + w.dgu);       // [P, 2f] = [dG | dU]
  int32_t* row_token = reinterpret_cast<int32_t*>(base + gw.row_token);
  float* row_w = reinterpret_cast<float*>(base + gw.row_w);
  bf16_t* act_w_ws = reinterpret_cast<bf16_t*>(base + gw.act_w);
  const bf16_t* act_w = a.act_w ? static_cast<const bf16_t*>(a.act_w) : act_w_ws;
  float* dw_partial = reinterpret_cast<float*>(base + gw.dw_partial);
  const bf16_t* G = static_cast<const bf16_t*>(a.g_save);
  const bf16_t* U = static_cast<const bf16_t*>(a.u_save);
  const WgradItems items = wgrad_items_at(a.ws, w, a.P, a.E);
  {
    ScheduleArgs sa{};
    sa.offsets = a.offsets; sa.E = a.E; sa.P = a.P; sa.bm = rt.bm; sa.rt = rt;
    sa.chunk_rows = wgrad_chunk_rows(a.P); sa.items = items;
    sa.pair_of_row = a.pair_of_row; sa.topk_w = a.topk_w; sa.T = a.T; sa.k = a.k; sa.row_token = row_token; sa.row_w = row_w;
    launch_schedules(sa, a.stream);
  }
  if (recompute) {
    bf16_t* Gr = reinterpret_cast<bf16_t*>(base + w.g);
    bf16_t* Ur = reinterpret_cast<bf16_t*>(base + w.u);
    launch_gate_up(a.x, a.w_gate, a.w_up, a.P, a.d, a.f, a.E, rt, Gr, Ur, nullptr, a.stream, row_token);
    G = Gr; U = Ur;
  }
  {  // dA = w (dy[token] Wd) with the SwiGLU derivative, the weight gradient's dot products and w * act
    RowArgs p{};
    p.a = static_cast<const bf16_t*>(a.dy); p.lda = a.d;
    p.w0 = static_cast<const bf16_t*>(a.w_down); p.w_expert_stride = static_cast<long>(a.d) * a.f; p.ldw = a.f;
    p.K = a.d; p.N = a.f; p.P = a.P; p.rt = rt;
    p.out0 = dgu; p.ldo = 2L * a.f; p.g = G; p.u = U;
    p.row_token = row_token; p.row_w = row_w; p.act_w = a.act_w ? nullptr : act_w_ws; p.dw_partial = dw_partial;
    if (p.act_w) launch_row<kDAct, true, true>(p, a.P, a.E, a.stream);
    else launch_row<kDAct, true, false>(p, a.P, a.E, a.stream);
  }
  launch_dx(dgu, a.w_gate, a.w_up, a.P, a.d, a.f, a.E, rt, a.dxp, a.stream);
  float* partial = reinterpret_cast<float*>(base + w.partial);
  WgradArgs down{}, gate_up{};
  {  // dWd[e] = dy[token]^T (w act)
    WgradArgs& p = down;
    p.lhs = static_cast<const bf16_t*>(a.dy); p.ld_lhs = a.d; p.M = a.d;
    p.rhs = act_w; p.ld_rhs = a.f; p.N = a.f;
    p.E = a.E; p.P = a.P; p.items = items; p.partial = partial;
    p.out0 = static_cast<bf16_t*>(a.dw_down); p.out1 = p.out0; p.m_split = a.d;
    p.row_token = row_token;
    p.dw_partial = dw_partial; p.dw_slots = dw_slots(rt, a.f); p.pair_of_row = a.pair_of_row; p.dtopk_w = a.dtopk_w;   // rides in the reduction launch
    launch_wgrad<0, true>(p, a.stream);
  }
  {  // [dWg[e]; dWu[e]] = [dG | dU]^T x[token]
    WgradArgs& p = gate_up;
    p.lhs = dgu; p.ld_lhs = 2L * a.f; p.M = 2 * a.f;
    p.rhs = static_cast<const bf16_t*>(a.x); p.ld_rhs = a.d; p.N = a.d;
    p.E = a.E; p.P = a.P; p.items = items; p.partial = partial + static_cast<size_t>(items.max_slots) * a.f * a.d;
    p.out0 = static_cast<bf16_t*>(a.dw_gate); p.out1 = static_cast<bf16_t*>(a.dw_up); p.m_split = a.f;
    p.row_token = row_token;
    launch_wgrad<1, true>(p, a.stream);
  }
  launch_wgrad_reduce("wgrad_reduce", down, &gate_up, a.stream);
}

// ============================================================================================
// Router linear (the gate that produces the logits) and its backward, on the same skeleton:
//   logits[T, E] (fp32)  = x[T, d] * Wr[E, d]^T          one segment of T rows, fp32 epilogue
//   dx[T, d]   (+)=  bf16(dz)[T, E] * Wr[E, d]           reduction over E, optional read-modify-write
//   dWr[E, d]       =  bf16(dz)[T, E]^T * x[T, d]         reduction over the T rows, chunked like the others
// The fp32 logit gradient is rounded to bf16 once for the two backward products (bf16 operands,
// fp32 accumulation, like every other product here).
// ============================================================================================
__global__ __launch_bounds__(256) void cast_f32_bf16_kernel(const float* __restrict__ in, bf16_t* __restrict__ out, long n8) {
  const long i = static_cast<long>(blockIdx.x) * 256 + threadIdx.x;
  if (i >= n8) return;
  float v[8];
  read8(in + i * 8, v);
  store16(out + i * 8, pack8(v));
}

struct RouterWs { size_t dz, partial, total; };
static int router_items(int T) { return std::max(1, ceil_div(T, router_chunk_rows(T))); }
static RouterWs router_ws(int T, int d, int E, bool bwd) {
  RouterWs w{};
  size_t off = 0;
  w.dz = off; w.partial = off;
  if (bwd) {
    off += align_up(static_cast<size_t>(T) * E * 2, 256);
    w.partial = off;
    off += align_up(static_cast<size_t>(router_items(T)) * E * d * sizeof(float), 256);
  }
  w.total = off + 256;
  return w;
}
size_t router_fwd_ws_bytes_bf16(int T, int d, int E) { return router_ws(T, d, E, false).total; }
size_t router_bwd_ws_bytes_bf16(int T, int d, int E) { return router_ws(T, d, E, true).total; }

void router_fwd_bf16(const RouterFwdArgs& a) {
  RowArgs p{};
  p.a = static_cast<const bf16_t*>(a.x); p.lda = a.d;
  p.w0 = static_cast<const bf16_t*>(a.w_router); p.w_expert_stride = 0; p.ldw = a.d;
  p.K = a.d; p.N = a.E; p.P = a.T;
  p.out_f32 = a.logits; p.ldo = a.E;
  launch_row_t<kRouterFwd, TileRouter>(p, a.T, 1, a.stream);
}

void router_bwd_bf16(const RouterBwdArgs& a) {
  const RouterWs w = router_ws(a.T, a.d, a.E, true);
  char* base = static_cast<char*>(a.ws);
  bf16_t* dz = reinterpret_cast<bf16_t*>(base + w.dz);
  const long n8 = static_cast<long>(a.T) * a.E / 8;
  MOE_LAUNCH("router_cast_dz", cast_f32_bf16_kernel, dim3(static_cast<unsigned>((n8 + 255) / 256)), dim3(256), 0, a.stream, a.dlogits, dz, n8);
  {  // dx (+)= dz * Wr
    RowArgs p{};
    p.a = dz; p.lda = a.E;
    p.w0 = static_cast<const bf16_t*>(a.w_router); p.w_expert_stride = 0; p.ldw = a.d;
    p.K = a.E; p.N = a.d; p.P = a.T;
    p.out0 = static_cast<bf16_t*>(a.dx); p.ldo = a.d; p.accumulate = a.accumulate;
    // A tile here is two slabs and an epilogue: while all tiles of 128 x 128 run at once they take 13-14 us where the few large
    // ones took 20-22 (300 and 1531 tokens, d = 2048; 4096, d = 1024); 8192 tokens, d = 2048, twice as many: 27.1 and 26.8.
    if (static_cast<long>(ceil_div(a.T, TileFew::BM)) * ceil_div(a.d, TileFew::BN) <= 2 * kCus) launch_row_t<kRouterDx, TileFew>(p, a.T, 1, a.stream);
    else launch_row_t<kRouterDx, TileBig>(p, a.T, 1, a.stream);
  }
  {  // dWr = dz^T x
    WgradArgs p{};
    p.lhs = dz; p.ld_lhs = a.E; p.M = a.E;
    p.rhs = static_cast<const bf16_t*>(a.x); p.ld_rhs = a.d; p.N = a.d;
    p.E = 1; p.P = a.T; p.partial = reinterpret_cast<float*>(base + w.partial);
    p.one_segment_items = router_items(a.T); p.chunk_rows = router_chunk_rows(a.T);
    p.out0 = static_cast<bf16_t*>(a.dw_router); p.out1 = p.out0; p.m_split = a.E;
    launch_wgrad<2>(p, a.stream);
    launch_wgrad_reduce("wgrad_router_reduce", p, nullptr, a.stream);
  }
}

// ============================================================================================
// Forward products with 8-bit block-scaled operands (same tiles, loaders, rings and way of walking the tiles)
// ============================================================================================
#include "gemm_mx8.inc"

}  // namespace moe
