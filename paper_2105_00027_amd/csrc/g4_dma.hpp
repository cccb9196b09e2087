// Copies straight from global memory into LDS, and waits for them, shared by
// the update kernels that stage their operands this way.
#pragma once

#include <hip/hip_runtime.h>

namespace g4 {
namespace upd {

typedef __attribute__((address_space(3))) unsigned char lds_t;

// global -> LDS, 16 bytes per lane: lane l copies base + off to LDS byte
// address lds + 16*l (base and lds wave-uniform).  Issued as inline assembly so
// that the compiler does not make LDS reads of the other buffer wait for these
// copies; the kernel waits for them itself (s_waitcnt before the barrier that
// publishes the buffer).  M0 carries the LDS address; one wait state separates
// its write from the copy.
__device__ __forceinline__ void dma16(const char *base, unsigned off, unsigned lds) {
    asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1"
                 :
                 : "v"(off), "s"(base), "s"(lds)
                 : "memory", "m0");
}

// Wait until at most n vector-memory operations of this wave are outstanding.
// n = 0 goes through the builtin so that the compiler knows every load of its
// own (the G(K2,K1) registers) has landed and adds no wait of its own later,
// where one would also wait for copies issued after this point.
__device__ __forceinline__ void wait_vm(int n) {
    if (n == 0) {
        __builtin_amdgcn_s_waitcnt(0);
        return;
    }
    switch (n) {
#define G4_W(k) case k: asm volatile("s_waitcnt vmcnt(" #k ")" ::: "memory"); break;
        G4_W(1) G4_W(2) G4_W(3) G4_W(4) G4_W(5) G4_W(6) G4_W(7) G4_W(8)
        G4_W(9) G4_W(10) G4_W(11) G4_W(12) G4_W(13) G4_W(14) G4_W(15) G4_W(16)
#undef G4_W
        default: asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); break;
    }
}

}  // namespace upd
}  // namespace g4
