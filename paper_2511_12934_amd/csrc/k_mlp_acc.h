// What the head kernels whose second layer accumulates in the accumulation registers share (k_mlp_acc.hip, k_mlp_acc3.hip).
#pragma once
#include "k_mfma.h"
#include "mfma_util.h"

namespace aif {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));

// What the end of a tile needs of its request.
struct AccOut {
    const int32_t *cand_ids;
    float *logits_out, *scores_out;
    int32_t n_cand, row_base;
};

// Layer 2's accumulators are the 256 accumulation registers, named by number.  The compiler, given 512-bit values to carry
// round the loops in them, copies and spills them; here it has vector registers only to manage, and every product is written out.
// It knows neither that these registers are taken (reserve_acc has them counted, no more) nor how long a product's result takes, so
// the build reads the assembly of the units that include this file and fails where the compiler uses an accumulation
// register or spills (into one), or puts an instruction of its own behind a product it must wait for (../asmcheck.py).
// The vector ALU reads a product's result behind two more products (64 cycles; it is there after 44).
__device__ __forceinline__ void mfma_v(f32x16 &c, const bf16x8 &a, const bf16x8 &b)
{
    asm volatile("v_mfma_f32_32x32x16_bf16 %0, %1, %2, %0" : "+v"(c) : "v"(a), "v"(b));
}
template <int LO> __device__ __forceinline__ void mfma_a(const bf16x8 &a, const bf16x8 &b)
{
    asm volatile("v_mfma_f32_32x32x16_bf16 a[%0:%1], %2, %3, a[%0:%1]" ::"n"(LO), "n"(LO + 15), "v"(a), "v"(b));
}
// two features through the ReLU into one word of the next layer's operand (written out: the compiler, which does not know
// where the values come from, would quiet them first)
__device__ __forceinline__ uint32_t relu_pair(float a, float b)
{
    uint32_t v;
    float t;
    asm volatile("v_max_f32 %0, 0, %2\n\tv_max_f32 %1, 0, %3\n\tv_cvt_pk_bf16_f32 %0, %0, %1" : "=&v"(v), "=&v"(t) : "v"(a), "v"(b));
    return v;
}
template <int R> __device__ __forceinline__ float acc_relu()
{
    float v;
    asm volatile("v_accvgpr_read_b32 %0, a[%1]\n\tv_max_f32 %0, 0, %0" : "=v"(v) : "n"(R));
    return v;
}
// two of them through the ReLU into one word of the next layer's operand
template <int R> __device__ __forceinline__ uint32_t acc_pair()
{
    uint32_t v;
    float t;
    asm volatile("v_accvgpr_read_b32 %0, a[%2]\n\tv_accvgpr_read_b32 %1, a[%3]\n\tv_max_f32 %0, 0, %0\n\tv_max_f32 %1, 0, %1\n\t"
                 "v_cvt_pk_bf16_f32 %0, %0, %1" : "=&v"(v), "=&v"(t) : "n"(R), "n"(R + 1));
    return v;
}
// four accumulation registers <- 16 bytes of LDS (waited for by hand at the stage's end)
template <int LO, int OFF> __device__ __forceinline__ void acc_from_lds(uint32_t addr)
{
    asm volatile("ds_read_b128 a[%0:%1], %2 offset:%3" ::"n"(LO), "n"(LO + 3), "v"(addr), "n"(OFF) : "memory");
}
__device__ __forceinline__ void reserve_acc()
{
    asm volatile("" :::
        "a0", "a1", "a2", "a3", "a4", "a5", "a6", "a7", "a8", "a9", "a10", "a11", "a12", "a13", "a14", "a15", "a16",
        "a17", "a18", "a19", "a20", "a21", "a22", "a23", "a24", "a25", "a26", "a27", "a28", "a29", "a30", "a31",
        "a32", "a33", "a34", "a35", "a36", "a37", "a38", "a39", "a40", "a41", "a42", "a43", "a44", "a45", "a46",
        "a47", "a48", "a49", "a50", "a51", "a52", "a53", "a54", "a55", "a56", "a57", "a58", "a59", "a60", "a61",
        "a62", "a63", "a64", "a65", "a66", "a67", "a68", "a69", "a70", "a71", "a72", "a73", "a74", "a75", "a76",
        "a77", "a78", "a79", "a80", "a81", "a82", "a83", "a84", "a85", "a86", "a87", "a88", "a89", "a90", "a91",
        "a92", "a93", "a94", "a95", "a96", "a97", "a98", "a99", "a100", "a101", "a102", "a103", "a104", "a105",
        "a106", "a107", "a108", "a109", "a110", "a111", "a112", "a113", "a114", "a115", "a116", "a117", "a118",
        "a119", "a120", "a121", "a122", "a123", "a124", "a125", "a126", "a127", "a128", "a129", "a130", "a131",
        "a132", "a133", "a134", "a135", "a136", "a137", "a138", "a139", "a140", "a141", "a142", "a143", "a144",
        "a145", "a146", "a147", "a148", "a149", "a150", "a151", "a152", "a153", "a154", "a155", "a156", "a157",
        "a158", "a159", "a160", "a161", "a162", "a163", "a164", "a165", "a166", "a167", "a168", "a169", "a170",
        "a171", "a172", "a173", "a174", "a175", "a176", "a177", "a178", "a179", "a180", "a181", "a182", "a183",
        "a184", "a185", "a186", "a187", "a188", "a189", "a190", "a191", "a192", "a193", "a194", "a195", "a196",
        "a197", "a198", "a199", "a200", "a201", "a202", "a203", "a204", "a205", "a206", "a207", "a208", "a209",
        "a210", "a211", "a212", "a213", "a214", "a215", "a216", "a217", "a218", "a219", "a220", "a221", "a222",
        "a223", "a224", "a225", "a226", "a227", "a228", "a229", "a230", "a231", "a232", "a233", "a234", "a235",
        "a236", "a237", "a238", "a239", "a240", "a241", "a242", "a243", "a244", "a245", "a246", "a247", "a248",
        "a249", "a250", "a251", "a252", "a253", "a254", "a255");
}

}  // namespace aif
