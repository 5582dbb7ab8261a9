// Key tiles of the latent layout (keys 576 wide, values their first 512
// columns) in LDS, and their loads: shared by the kernels over 64 and over 128
// query rows, both of four waves.
//
// A stage holds 32 keys: the first 512 columns, one row per 1 KB load, and
// after them the last 64 columns, eight rows per load: 36 loads, none for
// padding, nine a wave. At a row stride of 1056 bytes the operand reads of
// both products are free of bank conflicts; the 128-byte rows of the last
// columns are XOR-swizzled by 16-byte chunk, (row >> 1) & 7.
#pragma once

#include "device_common.h"
#include "kernels.h"

namespace flexattn {

typedef int32_t i32x4 __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) uint8_t* lds_byte_ptr;

constexpr int kLatentQK = 576, kLatentV = 512;
constexpr int kLatentBN = 32;                                  // keys of a tile
constexpr int kLatentRow = 1056;                               // LDS bytes from row to row
constexpr int kLatentTailOff = kLatentBN * kLatentRow;
constexpr int kLatentStage = kLatentTailOff + kLatentBN * 128;
constexpr int kLatentLoads = 9;                                // loads of a wave per tile

// Loads of a tile by wave w of four: its 8 rows lie in one page, so one
// resource on the page serves all nine, and two per-lane offsets are all that
// is held. Lane i of a row load takes 16-byte chunk i of the row (SWAP: i ^ 1
// in rows 16 to 31); of the tail load, chunk 64 + ((i & 7) ^ swizzle) of row
// i >> 3.
template <int P, bool SWAP>
struct LatentLoader {
  const uint8_t* kbase;
  uint32_t ksp, kss, ld_row, ld_tail, lds0;
  int w;

  __device__ __forceinline__ LatentLoader(const AttnParams& p, int head_kv, uint8_t* lds, int w_, int lane) : w(w_) {
    kbase = reinterpret_cast<const uint8_t*>(p.kc.base + int64_t(head_kv) * p.kc.sh);
    ksp = uint32_t(p.kc.sp) * 2u;
    kss = uint32_t(p.kc.ss) * 2u;
    ld_row = 16u * uint32_t(lane ^ (SWAP ? w >> 1 : 0));
    ld_tail = uint32_t(lane >> 3) * kss + 1024u + 16u * uint32_t((lane & 7) ^ (((8 * w + (lane >> 3)) >> 1) & 7));
    lds0 = uint32_t(reinterpret_cast<uintptr_t>((lds_byte_ptr)lds)) + uint32_t(8 * w) * kLatentRow;
  }

  // Resource of the wave's rows of the tile at key kb, in `page`. The record
  // count ends with the row of the last key before `end` (a whole row past
  // its start: the slot stride may be less than a row), so what is read past
  // it reads as zeros and touches no memory; a tile past `end` gets an empty
  // resource.
  __device__ __forceinline__ i32x4 source(int kb, int end, int page) const {
    const int g0 = kb + 8 * w;
    const uint64_t a = reinterpret_cast<uint64_t>(kbase + (uint64_t(uint32_t(page)) * ksp + uint32_t(g0 % P) * kss));
    const int rows = min(8, end - g0);
    i32x4 r = {__builtin_amdgcn_readfirstlane(int32_t(uint32_t(a))),
               __builtin_amdgcn_readfirstlane(int32_t(uint32_t(a >> 32) & 0xFFFFu)),
               __builtin_amdgcn_readfirstlane(rows > 0 ? int32_t(uint32_t(rows - 1) * kss + 2 * kLatentQK) : 0),
               kBufferFlags};
    // A vector instruction's scalar result needs 5 wait states before a
    // memory instruction reads it; the loads below are opaque to the compiler.
    asm volatile("s_nop 4" : "+s"(r));
    return r;
  }

  // Load j = 0 .. 8 of the wave into stage st.
  __device__ __forceinline__ void load_one(const i32x4& rsrc, int st, int j) const {
    const uint32_t dst = lds0 + uint32_t(st) * kLatentStage +
                         (j < 8 ? uint32_t(j) * kLatentRow : uint32_t(kLatentTailOff + w * 1024 - 8 * w * kLatentRow));
    const uint32_t off = j < 8 ? ld_row + uint32_t(j) * kss : ld_tail;
    asm volatile("s_nop 0\n\tbuffer_load_dwordx4 %0, %1, 0 offen lds" ::"v"(off), "s"(rsrc),
                 "{m0}"(__builtin_amdgcn_readfirstlane(dst))
                 : "memory");
  }
};

}  // namespace flexattn
