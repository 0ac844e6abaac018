// Loads from memory straight into LDS, written out (attn_fwd.hip).
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

namespace sc {

// N loads of 16 bytes per lane through a buffer resource over `bytes` bytes
// from `base`: load i of a wave fills the 1 KiB of LDS from byte address
// lds + 1024 i on with what its lanes' offsets voff[i] name (zeros past the
// end).  The second word of the resource holds address bits 32-47 and, above
// them, a stride of zero: the address as it is (device addresses have 48
// bits).
//
// The instruction takes the LDS address from M0 and needs one wait state
// after a scalar write of it.  Its resource must not have been written by a
// vector instruction (a readlane, as spilled scalar registers are restored)
// in the last five wait states, and the compiler's hazard pass does not look
// in here.  So the resource is put together by scalar moves, which wait for
// such a write by themselves and whose results the load may read at once;
// they also give M0 its wait state.  (Wait states alone, s_nop 3, cost more:
// a 24-token turn over 2048 13.06 us against 13.00, a chunked 40/8-head stack
// 1588 against 1584; without either they took 12.97 and 1580.)  The caller
// waits for the loads; there is no output register.
//
// The compiler keeps no value in M0 (it warns that the register is reserved),
// but may let two instructions share one write of it: hence the clobber.
#pragma clang diagnostic push
#pragma clang diagnostic ignored "-Winline-asm"
template <int N>
__device__ __forceinline__ void load_to_lds(uint32_t lds, const int (&voff)[N], uint64_t base, uint32_t bytes) {
  static_assert(N == 1 || N == 4, "one load, or four of one resource");
#define SC_LDS_RSRC              \
  "s_mov_b32 m0, %0\n\t"         \
  "s_mov_b64 s[96:97], %1\n\t"   \
  "s_mov_b32 s98, %2\n\t"        \
  "s_mov_b32 s99, 0x20000\n\t"
#define SC_LDS_LOAD(v) "buffer_load_dwordx4 " v ", s[96:99], 0 offen lds"
#define SC_LDS_NEXT "\n\ts_add_u32 m0, m0, 0x400\n\ts_nop 0\n\t"
  if constexpr (N == 1)
    asm volatile(SC_LDS_RSRC SC_LDS_LOAD("%3")
                 :
                 : "s"(lds), "s"(base), "s"(bytes), "v"(voff[0])
                 : "memory", "m0", "s96", "s97", "s98", "s99");
  else
    asm volatile(SC_LDS_RSRC SC_LDS_LOAD("%3") SC_LDS_NEXT SC_LDS_LOAD("%4") SC_LDS_NEXT SC_LDS_LOAD("%5")
                     SC_LDS_NEXT SC_LDS_LOAD("%6")
                 :
                 : "s"(lds), "s"(base), "s"(bytes), "v"(voff[0]), "v"(voff[1]), "v"(voff[2]), "v"(voff[3])
                 : "memory", "m0", "scc", "s96", "s97", "s98", "s99");
#undef SC_LDS_RSRC
#undef SC_LDS_LOAD
#undef SC_LDS_NEXT
}
#pragma clang diagnostic pop

}  // namespace sc
