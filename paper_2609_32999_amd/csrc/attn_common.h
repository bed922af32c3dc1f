// Device definitions shared by the bf16 attention kernels (attn.hip,
// attn_pipe.hip): MFMA operand types, the LDS tile layouts and the
// direct global->LDS load.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

namespace tsr {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));
typedef _Float16 f16x2 __attribute__((ext_vector_type(2)));
typedef float f32x16 __attribute__((ext_vector_type(16)));

union Frag {
  uint4 u;
  uint32_t w[4];
  bf16x8 b;
  f16x8 h;
  f16x2 p[4];
};

constexpr int kD = 128;
// Keys per tile of the bf16 kernels.
constexpr int kKT = 32;
// V^T rows (fp16) are 16-byte aligned and hold each 16-key step permuted as
// keys [0..3, 8..11, 4..7, 12..15], so that the eight keys a lane feeds to
// the PV MFMA (4h .. 4h+3 and 8+4h .. 8+4h+3 for half-wave h, the order in
// which the S^T accumulators hand out P^T) are one 16-byte LDS read.
constexpr int kVStr = kKT + 8;         // fp16 elements per V^T row in LDS
// A K tile sits in LDS in 1 KB blocks in fragment order: a direct
// global->LDS load of 16 bytes per lane fills one block, and fragment reads
// are contiguous runs at immediate offsets (no bank conflicts).  In the
// pipelined kernel a block is a 16-dim step kst of the QK^T MFMAs, lane l's 16
// bytes (at l * 16) being K[l % 32][16 kst + 8 (l / 32) .. + 8]; the row-block
// kernel's order is in attn.hip.
constexpr int kKBlk = 1024;
constexpr int kKBytes = 8 * kKBlk;
constexpr int kVBytes = kD * kVStr * 2;
// s_waitcnt immediate that waits for every outstanding vector memory
// access (direct global->LDS loads included) and leaves the other counters.
constexpr int kWaitVm0 = 0x0F70;
// Lazy rescale threshold (log2 units): P may grow to 2^kLazy before the
// running max is moved.
constexpr float kLazy = 8.0f;
constexpr float kLazySum = 256.0f;   // 2^kLazy

// Position of key k (0 .. 31) of a tile in its permuted V^T row.
__device__ __forceinline__ int vt_col(int k) {
  const int b = k >> 4, kk = k & 15;
  return 16 * b + ((kk >> 2) & 1) * 8 + ((kk >> 3) & 1) * 4 + (kk & 3);
}

// Direct global->LDS load of 16 bytes per lane: lane l's bytes land at LDS
// address lds + 16 l (lds wave-uniform).  Written as assembly so that the
// compiler does not take the LDS write for a possible alias of the LDS reads
// that follow it (it would wait for the load before each of them); callers
// wait for these loads themselves (s_waitcnt vmcnt) before the barrier that
// hands the buffer to the workgroup.  M0 holds no other value in the
// kernels that use this.
#pragma clang diagnostic push
#pragma clang diagnostic ignored "-Winline-asm"
__device__ __forceinline__ void lds_dma16(const void* src, uint32_t lds) {
  asm volatile("s_mov_b32 m0, %1\n\tglobal_load_lds_dwordx4 %0, off"
               :: "v"(src), "s"(lds) : "m0");
}
// The same from a wave-uniform address plus a 32-bit lane offset in bytes
// plus OFS: one address register a lane instead of two, no 64-bit adds.  The
// instruction adds its offset to the LDS address too, hence the lds - OFS.
template <int OFS>
__device__ __forceinline__ void lds_dma16(const void* base, uint32_t off, uint32_t lds) {
  asm volatile("s_mov_b32 m0, %2\n\tglobal_load_lds_dwordx4 %0, %1 offset:%3"
               :: "v"(off), "s"(base), "s"(lds - OFS), "n"(OFS) : "m0");
}
#pragma clang diagnostic pop

// One wave's normalized output rows (the O^T accumulators: lane l holds row
// l % 32, dims 32 db + 8 rg + 4 (l / 32) .. + 3 in o[db][4 rg ..]) as bf16 to
// out rows of kD elements, through kOutLds bytes of LDS that are the wave's
// own.  Stored from the accumulators, an instruction touches 32 rows 16 bytes
// at a time; from LDS it writes 64 bytes of each of 16 rows, half the lines
// for the same bytes.  RAG-8B LOCAL attention 251 -> 243 us, GLOBAL 563 -> 557,
// agent memory 1,630 -> 1,614, fp8 RAG 1,649 -> 1,620; outputs keep their bits.
// row_off(r): element offset of row r in out; rows r < n are stored.
constexpr int kOutStr = 80;                      // bytes per row of a 32-dim block
constexpr int kOutLds = 32 * kOutStr;
template <typename RowOff>
__device__ __forceinline__ void store_out(const f32x16 (&o)[4], float inv, uint8_t* lds,
                                          int lane, int n, uint16_t* __restrict__ out,
                                          RowOff row_off) {
  typedef uint32_t lds2 __attribute__((ext_vector_type(2), may_alias));
  typedef uint32_t lds4 __attribute__((ext_vector_type(4), may_alias));
  const int lrow = lane & 31, lh = lane >> 5, r4 = lane >> 2, c4 = lane & 3;
  const int64_t off[2] = {row_off(min(r4, n - 1)), row_off(min(r4 + 16, n - 1))};
#pragma unroll
  for (int db = 0; db < 4; ++db) {
#pragma unroll
    for (int rg = 0; rg < 4; ++rg) {
      typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
      const bf16x4 v = {(__bf16)(o[db][4 * rg] * inv), (__bf16)(o[db][4 * rg + 1] * inv),
                        (__bf16)(o[db][4 * rg + 2] * inv), (__bf16)(o[db][4 * rg + 3] * inv)};
      *reinterpret_cast<lds2*>(lds + lrow * kOutStr + 16 * rg + 8 * lh) =
          __builtin_bit_cast(lds2, v);
    }
    // LDS keeps a wave's accesses in order; this keeps the compiler to it
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const lds4 v = *reinterpret_cast<const lds4*>(lds + (r4 + 16 * h) * kOutStr + 16 * c4);
      if (r4 + 16 * h < n) *reinterpret_cast<lds4*>(out + off[h] + 32 * db + 8 * c4) = v;
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
  }
}

__device__ __forceinline__ uint32_t lds_addr(const void* p) {
  return (uint32_t)(uintptr_t)(__attribute__((address_space(3))) const void*)p;
}

}  // namespace tsr
