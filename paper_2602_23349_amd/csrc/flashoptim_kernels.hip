// FlashOptim device code for gfx950 (MI355X): the fused optimizer-step kernels
// (paper Algorithms 4, 5, 6), the standalone codecs (Algorithms 1, 2, 3) and the
// checkpoint gather/scatter copy.
//
// Numerical contract.  Every floating-point operation is one IEEE binary32
// operation (round-to-nearest-even, subnormals kept).  This file must be built
// with -ffp-contract=off and correctly rounded division / square root (hipcc's
// default), because 8-bit codes and correction bytes are compared bit for bit
// against an independent CPU implementation of the same algorithms.
// One exception, selected by the EXACT template flag of the AdamW step: with EXACT = false
// (the default entry point) the quotient m_hat / (sqrt(v_hat) + eps) is faithfully rounded
// (within one ulp of the correctly rounded value, and equal to it for all but about one operand
// pair in 10^9); the state codes and scales are unaffected, the master weight can differ by one ulp.
//
// The step is bandwidth-bound by definition (12.25 algorithmic bytes per parameter
// for AdamW), but an exactly rounded body, written down as the definitions have it, costs
// well over a hundred VALU instructions per parameter, which at 8 TB/s is more than the chip's
// non-packed FP32 rate admits.  The design choices below are about keeping VALU work per
// element low without changing a single rounding (AdamW: 64 to 68 instructions per element):
//   * decoding a code is a function of one byte: rho/127 and phi_m^-1(code/127) come from two 256-entry LDS
//     tables that each workgroup fills once with the results of the IEEE divisions that define them; code/255 is
//     the code times the reciprocal as the sum of two floats, the IEEE quotient for every byte;
//   * the 2^l scalings of Algorithm 1 are floats made of the exponent bits of theta', one or two integer
//     operations each (wavefronts with a weight below 2^-110, zeros included, take a general form);
//   * Round(x) to an 8-bit integer is one FP32 addition of 1.5 * 2^23, whose low
//     mantissa byte is the round-half-even integer in two's complement;
//   * BF16 rounding uses the hardware v_cvt_pk_bf16_f32 (two elements per issue);
//   * an 8-bit state code is Round(y) of a value y whose exact evaluation needs an IEEE
//     division (momentum) or square root (variance).  The kernel evaluates y with the 1-ulp hardware
//     reciprocal / with the square root it already has from the update; that estimate provably
//     differs from the exact y by less than a small w.  It rounds estimate - w and estimate + w
//     (v_cvt_pk_u8_f32: round-half-even, saturation and byte packing in one instruction); where both
//     give the same integer the code is decided.  Only when they differ for some lane of the
//     wavefront (a few percent of the wavefronts) are the four elements concerned recomputed with
//     the exact sequence.  Codes are bit-identical to the exact evaluation in every case;
//   * sqrt(v_hat) and m_hat / (sqrt(v_hat) + eps) use the 1-ulp hardware reciprocal square
//     root / reciprocal followed by FMA residual corrections that yield the correctly rounded
//     result for operands inside a stated range (the square root: verified for every value of
//     the range by the device self-test; the division: by the argument beside div_rn_midrange, from
//     a property of the reciprocal that the self-test checks); a wave-uniform range test selects the
//     general sequence otherwise.  With EXACT = false the division takes one residual correction of
//     the unrefined quotient (div_faithful).
//
// Work decomposition.  A lane owns 8 consecutive elements per tile: BF16 streams move as
// 128-bit and byte streams as 64-bit accesses, and a quantisation group (32 elements) is a
// lane quad, so the group absmax needs two DPP quad permutes and no LDS.  A workgroup (256
// lanes; 512 for SGD and Lion over 2^27 elements and more) handles one tile of consecutive elements of one
// tensor; a small two-level table maps the workgroup index to (tensor, tile) so that one call covers a
// whole parameter list, issued as a few consecutive launches.  Stream addresses are a scalar 64-bit
// tile base plus a 32-bit lane offset.  A lane owns 4 elements, and a group is 8 lanes, where FP32 streams are
// moved (ablation variants, codecs, conversions: a 128-bit FP32 access per lane then covers whole cache lines)
// and where a launch is small (fewer than 2^20 elements: more wavefronts, each with half the work).  Where a workgroup
// shares nothing (plain FP32 steps, split and reconstruct, large compressions) it is a single wavefront.  Large launches hold
// fewer workgroups to a compute unit than fit (step_resident) and store past the caches (step_through).

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

#include "flashoptim_device.h"

namespace fo {

// A launch.  (Through hipLaunchKernel itself: with <<<>>> the host takes 0.15-0.2 us more of the 3 that a launch costs it.)
template <typename... P>
static hipError_t launch(void (*kernel)(P...), unsigned blocks, unsigned threads, unsigned lds, hipStream_t s,
                         const std::decay_t<P>&... p) {
    void* args[] = {const_cast<void*>(static_cast<const void*>(&p))...};
    return hipLaunchKernel(reinterpret_cast<const void*>(kernel), dim3(blocks), dim3(threads), args, lds, s);
}

typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
typedef float floatx2_t __attribute__((ext_vector_type(2)));

// ------------------------------------------------------------------ helpers --

typedef uint32_t u32x4_t __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2_t __attribute__((ext_vector_type(2)));

// 128-bit global accesses of the streaming data (each byte is touched once per step).
__device__ __forceinline__ uint4 ld128(const void* p) {
    const u32x4_t v = __builtin_nontemporal_load(reinterpret_cast<const u32x4_t*>(p));
    return make_uint4(v.x, v.y, v.z, v.w);
}
__device__ __forceinline__ void st128(void* p, uint32_t a, uint32_t b, uint32_t c, uint32_t d) {
    const u32x4_t v = {a, b, c, d};
    __builtin_nontemporal_store(v, reinterpret_cast<u32x4_t*>(p));
}

__device__ __forceinline__ float u2f(uint32_t u) { return __uint_as_float(u); }
__device__ __forceinline__ uint32_t f2u(float f) { return __float_as_uint(f); }

// Maximum over the lanes that share a 32-element group: a lane quad (8 elements per lane) or two quads (4 per lane).  Each step is ONE instruction, v_max_f32 with its first operand taken
// from the neighbouring lane through a DPP quad permute (written as inline assembly: from the
// builtin the compiler makes a DPP move, two canonicalising maxima and the maximum itself).  The
// s_nop covers the two wait states a DPP read needs after the instruction that wrote its source.
// v_max_f32 returns the other operand when one is NaN, like fmaxf.
__device__ __forceinline__ float max_across_lane_pair(float x) {
    float r;
    asm("s_nop 1\n\tv_max_f32_dpp %0, %1, %1 quad_perm:[1,0,3,2] row_mask:0xf bank_mask:0xf" : "=v"(r) : "v"(x));
    return r;
}
__device__ __forceinline__ float max_across_pair_of_pairs(float x) {
    float r;
    asm("s_nop 1\n\tv_max_f32_dpp %0, %1, %1 quad_perm:[2,3,0,1] row_mask:0xf bank_mask:0xf" : "=v"(r) : "v"(x));
    return r;
}
// After the first two steps the four lanes of a quad agree, so mirroring each run of eight lanes brings every
// lane the other quad's value.
__device__ __forceinline__ float max_across_two_quads(float x) {
    float r;
    asm("s_nop 1\n\tv_max_f32_dpp %0, %1, %1 row_half_mirror row_mask:0xf bank_mask:0xf" : "=v"(r) : "v"(x));
    return r;
}
template <int VEC>
__device__ __forceinline__ float group_max(float x) {
    static_assert(VEC == 4 || VEC == 8, "lanes per group: 8 or 4");
    x = max_across_pair_of_pairs(max_across_lane_pair(x));
    if (VEC == 4) x = max_across_two_quads(x);
    return x;
}

// Round-half-even of y (|y| <= 2^21) to an integer, returned in two's complement in the
// low bits of the result.
__device__ __forceinline__ uint32_t round_to_int_bits(float y) { return f2u(y + 12582912.0f); }

// log2 of half the BF16 ULP of the value whose BF16 bit pattern is `b` (Algorithm 1:
// l = floor(log2 ULP(theta')) - 1).  Zero and subnormals use the lowest binade's spacing.
__device__ __forceinline__ int half_ulp_log2(uint32_t b) {
    int E = (int)((b >> 7) & 0xffu);
    E = E < 1 ? 1 : E;
    return E - 135;
}

// BF16 round-to-nearest-even of two floats: a in the low half, b in the high half.
__device__ __forceinline__ uint32_t bf16_pack(float a, float b) {
    floatx2_t f = {a, b};
    bf16x2_t r = __builtin_convertvector(f, bf16x2_t);
    return __builtin_bit_cast(uint32_t, r);
}

// Reciprocal of an FP16 scale, formed as hardware estimate + one Newton step.  The argument takes
// only the 31,743 positive finite FP16 values; for every one of them this sequence returns the
// correctly rounded 1/s (checked exhaustively on the device by flashoptim_selftest).
__device__ __forceinline__ float recip_of_fp16(float s) {
    const float r0 = __builtin_amdgcn_rcpf(s);
    const float e = fmaf(-s, r0, 1.0f);
    return fmaf(e, r0, r0);
}
// FP16 scale of a group from its FP32 absmax: saturate at 65504, round to nearest even.
// Returns the FP16 bits; *s is the scale as the decoder will read it.
__device__ __forceinline__ uint32_t group_scale(float absmax, float* s) {
    const float a = fminf(absmax, 65504.0f);
    const _Float16 h = (_Float16)a;
    *s = (float)h;
    return (uint32_t)__builtin_bit_cast(uint16_t, h);
}
// The correctly rounded reciprocal of a group's scale; 0 when the scale is 0, so that every code of the group becomes 0.
__device__ __forceinline__ float recip_of_scale(float s) { return (s == 0.0f) ? 0.0f : recip_of_fp16(s); }

// Correctly rounded square root for 2^-96 <= x <= FLT_MAX: the hardware reciprocal-square-root
// estimate (1 ulp) and one Newton correction, each step one FMA.  That this sequence returns the
// correctly rounded root for EVERY FP32 value of that range is a property of the hardware estimate
// which is verified exhaustively on the device (all 1,879,048,192 values): ahead of the first AdamW
// step on a device (until that check has passed, the device word behind StepConsts::sqrt_min holds +inf
// and the kernels use sqrtf) and by flashoptim_selftest.  Below
// 2^-96 the residual x - s*s leaves the normal range and the result is only within one ulp; zero,
// infinity and NaN give NaN.  Callers check the range and use sqrtf() otherwise.
__device__ __forceinline__ float sqrt_rn_midrange(float x) {
    const float y = __builtin_amdgcn_rsqf(x);
    const float s = x * y, h = 0.5f * y;
    return fmaf(fmaf(-s, s, x), h, s);
}
// Correctly rounded n / d for operands well inside the normal range: 2^-60 <= |n|, d <= 2^60 (no intermediate result
// leaves the normal range, so the range scaling and the special-case fix-up of the general division are not needed;
// callers check the range).  Every step after the hardware reciprocal r0 (1 ulp) is one FMA or one product:
//   e = 1 - d r0;  q1 = q0 + q0 e with q0 = n r0;  r1 = r0 + r0 e;  result q1 + (n - d q1) r1.
// Why that is RN(n / d).  (1) r1 is the correctly rounded reciprocal: a property of the hardware estimate, which
// scales with the exponent and holds for every mantissa (flashoptim_selftest, section 1).  (2) q0 e removes the error of
// r0 down to its square (2^-46), so what separates q1 from n / d is the rounding of q0 and its own: at most one ulp
// (plus 2^-22).  Hence n - d q1 is exact, and before the last rounding the result is off by |n / d - q1| |d r1 - 1|.
// (3) With the mantissas of n and d as integers of 24 bits, n / d is never the middle of two FP32 numbers, and is at
// least 2^-24 / b ulp away from one, b in [1, 2) being the mantissa of d.  Near a middle |n / d - q1| is half an
// ulp, so by (1) the error is below 0.5 b 2^-25 < 2^-24 / b ulp, as b < 2: it cannot change the rounding.
// (The classical form refines r first and corrects the quotient twice: one instruction more per element.)
__device__ __forceinline__ float div_rn_midrange(float n, float d) {
    const float r0 = __builtin_amdgcn_rcpf(d);
    const float e = fmaf(-d, r0, 1.0f);
    const float q0 = n * r0;
    const float q1 = fmaf(q0, e, q0);
    const float r1 = fmaf(e, r0, r0);
    return fmaf(fmaf(-d, q1, n), r1, q1);
}

// Faithful division: one residual correction of the quotient formed with the 1-ulp hardware reciprocal,
// each step one FMA.  The value before the final rounding is within 2^-23 ulp of the exact quotient, so the
// result is the correctly rounded one except when the exact quotient lies that close to the middle between
// two FP32 numbers; then it is the other neighbour (the device self-test bounds the difference to one ulp and
// counts such operand pairs: 52 among 2^36 random pairs on MI355X, 7.6e-10).  Denominator range as for
// div_rn_midrange.  A numerator below 2^-60 is admitted: down to 2^-103 nothing changes; below that the
// residual can leave the normal range and the error can reach a few ulp of a quotient smaller than 2^-43.
__device__ __forceinline__ float div_faithful(float n, float d) {
    const float r = __builtin_amdgcn_rcpf(d);
    const float q = n * r;
    return fmaf(fmaf(-d, q, n), r, q);
}

// Exact Q_m code (low byte of the result) of one element given the reciprocal group scale
// (Algorithm 2, encoder).
__device__ __forceinline__ uint32_t m_code_exact(float m, float r) {
    const float m1 = m * r;
    const float num = 2.0f * m1;
    const float den = 1.0f + fabsf(m1);
    const float m2 = num / den;
    const float y = __builtin_amdgcn_fmed3f(m2 * 127.0f, -127.0f, 127.0f);
    return round_to_int_bits(y);
}

// The same code decided from an estimate.  m1 and den are formed exactly as above; the quotient uses v_rcp_f32 (1 ulp), so
// 254 * (m1 * rc) differs from the exact y by at most (2 + 1 + 1) * 2^-24 * 128 < 3.1e-5 wherever the clamp is not active.
// p = m1 * rc + 1/2 is one fused multiply-add, whose rounding (half an ulp of a value below 1, times 254) adds 7.6e-6 and
// whose clamp to [0, 1] costs nothing.  The function returns y* + 128 -+ w = 254 p + (1 -+ w), each ONE fused multiply-add
// (half an ulp of a value below 256: 7.7e-6): if both round to the same integer no rounding tie lies within 4.7e-5 of y* on
// either side and that integer is the exact code plus 128.  The integers come from v_cvt_pk_u8_f32 (round-half-even,
// saturating at 0 and 255, one byte of a word per instruction): its saturation at 255 is the upper clamp of the code (+127);
// the lower clamp (-127) is the clamp of p at 0.
constexpr float kTieWindowM = 6.0e-5f;
__device__ __forceinline__ void m_code_bracket(float m, float r, float* lo, float* hi) {
    const float m1 = m * r;
    const float den = 1.0f + fabsf(m1);
    const float rc = __builtin_amdgcn_rcpf(den);
    const float p = __builtin_amdgcn_fmed3f(fmaf(m1, rc, 0.5f), 0.0f, 1.0f);
    *lo = fmaf(p, 254.0f, 1.0f - kTieWindowM);
    *hi = fmaf(p, 254.0f, 1.0f + kTieWindowM);
}

// Exact Q_v code of one element from v and the reciprocal group scale (Algorithm 3, encoder).
__device__ __forceinline__ uint32_t v_code_exact(float v, float r) {
    const float y = __builtin_amdgcn_fmed3f((sqrtf(v) * r) * 255.0f, 0.0f, 255.0f);
    return round_to_int_bits(y);
}

// The same value when v is known to be inside the range of sqrt_rn_midrange.
__device__ __forceinline__ uint32_t v_code_exact_midrange(float v, float r) {
    const float y = __builtin_amdgcn_fmed3f((sqrt_rn_midrange(v) * r) * 255.0f, 0.0f, 255.0f);
    return round_to_int_bits(y);
}

// The same code decided from root_hat = sqrt(v * rbc2) (exactly rounded, already computed for the update)
// and kr255 = 255 * sqrt(1 / rbc2) * r, formed per group to within one rounding (the host passes the constant
// in two halves).  Relative errors of y* = root_hat * kr255 against the exact argument y of Round(), in units
// of 2^-24: the rounding of v * rbc2 (1/2 after the root), of the root (1), of kr255 (1), against the three
// roundings of the exact chain sqrt, * r, * 255 (3): 5.5 * 2^-24 * 255.5 < 8.4e-5 in y below the saturation
// point.  The function returns y* -+ w, each ONE fused multiply-add (rounding: half an ulp of a value below
// 256, 7.7e-6): if both round to the same integer no rounding tie lies within 9.2e-5 of y*, and that integer
// is the exact code.  The conversion's saturation at 255 is the clamp of Algorithm 3.
constexpr float kTieWindowV = 1.0e-4f;
__device__ __forceinline__ void v_code_bracket(float root_hat, float kr255, float* lo, float* hi) {
    *lo = fmaf(root_hat, kr255, -kTieWindowV);
    *hi = fmaf(root_hat, kr255, kTieWindowV);
}
// Round-half-even of x to 0..255 (saturating; NaN gives 0), placed in byte `k` of `word`.
__device__ __forceinline__ uint32_t put_u8(float x, uint32_t k, uint32_t word) {
    return __builtin_amdgcn_cvt_pk_u8_f32(x, k, word);
}

// Low bytes of four words -> one word (c0 in byte 0).
__device__ __forceinline__ uint32_t pack_low_bytes(uint32_t c0, uint32_t c1, uint32_t c2, uint32_t c3) {
    const uint32_t t01 = __builtin_amdgcn_perm(c1, c0, 0x0c0c0400u);
    const uint32_t t23 = __builtin_amdgcn_perm(c3, c2, 0x0c0c0400u);
    return __builtin_amdgcn_perm(t23, t01, 0x05040100u);
}

__device__ __forceinline__ bool any_lane(bool p) { return __builtin_amdgcn_ballot_w64(p) != 0; }

// ------------------------------------------------------------- decode tables --

struct DecodeTables {
    float rho[256];    // (float)(int8)i / 127
    float m[256];      // phi_m^-1((float)(int8)i / 127)
    float v[256];      // (float)i / 255
};

// All tables are compile-time constants.  The compiler evaluates constant expressions in
// IEEE binary32 with round-to-nearest-even, so every entry is the result of the same single
// divisions the definitions prescribe (the decoders of Algorithms 1, 2 and 3).
constexpr DecodeTables make_decode_tables() {
    DecodeTables t{};
    for (int i = 0; i < 256; ++i) {
        const int sb = i < 128 ? i : i - 256;
        const float z = (float)sb / 127.0f;
        const float az = z < 0.0f ? -z : z;
        t.rho[i] = z;
        t.m[i] = z / (2.0f - az);
        t.v[i] = (float)i / 255.0f;
    }
    return t;
}
__device__ const DecodeTables g_decode_tables = make_decode_tables();

// i / 127 of a signed and i / 255 of an unsigned byte, correctly rounded: the reciprocal as the sum of two floats, of which
// the product with i needs one rounding each.  That this is the IEEE quotient for all 256 bytes is a matter of trying them.
__device__ __forceinline__ float code_over_127(uint32_t byte) {
    const float i = (float)(int8_t)byte;
    return fmaf(i, 0x1.020408p-7f, i * 0x1.020408p-35f);
}
__device__ __forceinline__ float code_over_255(uint32_t byte) {
    const float i = (float)byte;
    return fmaf(i, 0x1.010102p-8f, i * -0x1.fdfdfep-33f);
}

// A step's workgroup stages the tables that its variant reads (up to 2 KB, L2-resident) into LDS: rho (SPLIT) and m
// (QUANT).  256 lanes load an entry of each; of 512, the lower half loads rho, the upper m.  The staging is split into its load half
// and its store half so that a kernel can issue the loads first of all (they depend on nothing) and store to LDS only after it has
// issued its streaming loads.
//   The variance's factor is formed from its code (code_over_255): three instructions where the look-up takes one and an LDS read, of
// which two thirds of the cycles are bank conflicts, and the large AdamW steps are bound by the package's power.  Looked up -> formed, us: four
// Llama layers with embedding and head 3871 -> 3822, 3830 -> 3810 and, with the changes just before it, 3874 -> 3858 on three cards, the last
// within what two runs differ by; a layer by release 450 -> 449, ResNet-50 54.6 -> 53.8, state
// quantisation only 490 -> 486, 12 M 26.2 -> 25.6, 4 M 8.69 -> 8.58, 2 M 5.84 -> 5.77.  The same for rho, after that, gains 0.5 % in large
// Lion steps (GPT-2 192.4 -> 191.5) and loses elsewhere: four layers 3769 -> 3788, AdamW over 4 M 8.66 -> 8.91, SGD over 5 M 8.97 -> 9.78.
struct StepTables {
    float rho_scaled[256];    // rho / 127 * 2^-8 (exact), see reconstruct_fast
    float m[256];
};
struct TableEntries {
    float rho, m;
};
template <int THREADS, bool SPLIT, bool QUANT>
__device__ __forceinline__ void load_table_entries(TableEntries& e, int tid) {
    static_assert(THREADS == 256 || THREADS == 512, "");
    // scalar base + 32-bit lane offset, so that no 64-bit address arithmetic lands on the vector ALU
    typedef const __attribute__((address_space(1))) uint8_t* base_t;
    typedef const __attribute__((address_space(1))) float* fptr_t;
    const base_t base = (base_t)&g_decode_tables;
    const uint32_t o4 = (uint32_t)(tid & 255) * 4u;
    if (SPLIT && (THREADS == 256 || tid < 256)) e.rho = *(fptr_t)(base + offsetof(DecodeTables, rho) + o4);
    if (QUANT && (THREADS == 256 || tid >= 256)) e.m = *(fptr_t)(base + offsetof(DecodeTables, m) + o4);
}
template <int THREADS, bool SPLIT, bool QUANT>
__device__ __forceinline__ void store_table_entries(StepTables& t, const TableEntries& e, int tid) {
    const int i = tid & 255;
    if (SPLIT && (THREADS == 256 || tid < 256)) t.rho_scaled[i] = e.rho * 0.00390625f;
    if (QUANT && (THREADS == 256 || tid >= 256)) t.m[i] = e.m;
}

// In-kernel forms of C^-1 and of the rho half of C (Algorithm 1).  E is the exponent field of theta', 2^l half the BF16
// ULP of theta' (l = E - 135 for E >= 1), q = rho / 127; `base` and `t` are theta' as FP32.
//   C^-1: theta_hat = theta' + q * 2^l, the product rounded if it is subnormal (what the two-factor form in Algorithm 1's
//         decoder does).  With the exponent field of theta' as a float of its own, 2^(E-127), and q * 2^-8 from the table,
//         the product is the same one; it is exact, and one fused multiply-add gives the sum, if E >= 16.
//   C:    rho = Round(e_norm * 127) with e_norm = e * 2^-l.  127 * 2^-l is a float for 15 <= E: its bits follow from those
//         of theta' by one subtraction.  e has at most 16 significant bits below theta', so e * (127 * 2^-l) is exact, and
//         adding the rounding constant inside the fused multiply-add rounds the value that Round() would.  For a finite
//         theta' the clamp of Algorithm 1 is the identity (|e| <= 2^l under round-to-nearest); for theta' = +-inf the
//         product is +-inf or NaN and the low byte of (+-inf or NaN) + 1.5 * 2^23 is 0.
// Callers take these forms where every weight of the wavefront has a magnitude of at least kSplitFastLo = 2^-110, hence
// E >= 16, before and after the update; otherwise (zero weights, above all) the general forms below, with the same bits
// where both apply.  A theta' of +-inf passes only with a rho that leaves it infinite: 0 * inf and inf - inf are NaN, which
// the test refuses.
// (These took tables of 2^l and of the encoder's two factors, indexed by E: two look-ups and two instructions more per element.)
constexpr float kSplitFastLo = 7.703719777548943e-34f;    // 2^-110
__device__ __forceinline__ float reconstruct_fast(float base, float q_scaled) {
    return fmaf(q_scaled, u2f(f2u(base) & 0x7f800000u), base);
}
__device__ __forceinline__ float reconstruct_general(float base, float q_scaled) {
    const int E = (int)((f2u(base) >> 23) & 0xffu);
    return base + ldexpf(q_scaled, (E < 1 ? 1 : E) - 127);
}
__device__ __forceinline__ uint32_t rho_bits_fast(float theta, float t) {
    const float scale = u2f(0x867e0000u - (f2u(t) & 0x7f800000u));     // 127 * 2^(135 - E)
    return f2u(fmaf(theta - t, scale, 12582912.0f));
}
__device__ __forceinline__ uint32_t rho_bits_general(float theta, float t) {
    const int E = (int)((f2u(t) >> 23) & 0xffu);
    const float y = ldexpf(theta - t, 135 - (E < 1 ? 1 : E)) * 127.0f;
    return E == 255 ? 0u : round_to_int_bits(y);
}
// Minimum that is NaN if either operand is (one v_minimum3_f32 for two of them).
__device__ __forceinline__ float min_or_nan(float a, float b) { return __builtin_elementwise_minimum(a, b); }

// -------------------------------------------------------------- lane vectors --
//
// VEC consecutive elements per lane: 8 (the byte streams move as 64-bit accesses, a group is a lane quad) or 4 (32-bit
// accesses, a group is eight lanes).  With 16 every stream would move as 128-bit accesses, but a lane's BF16 data would
// be two of them that each cover half of every line, and fewer wavefronts fit on a SIMD.

template <int VEC>
struct LaneIO {
    uint32_t p[VEC / 2];    // VEC BF16 theta'
    uint32_t g[VEC / 2];    // VEC BF16 gradients
    uint32_t r[VEC / 4];    // VEC INT8 rho
    uint32_t mq[VEC / 4];   // VEC INT8 momentum codes
    uint32_t vq[VEC / 4];   // VEC UINT8 variance codes
    uint32_t ms, vs;        // FP16 scale bits of the lane's group
    // uncompressed halves (ablation variants only; dead otherwise)
    float th32[VEC];        // FP32 master weights when weights are not split
    float m32[VEC];         // FP32 momentum when states are not quantized
    float v32[VEC];         // FP32 variance when states are not quantized
};

// Streaming accesses of a full lane.  Every stream of a tile is addressed as a wave-uniform
// 64-bit base (tensor pointer + tile offset, kept in scalar registers) plus a 32-bit byte offset
// of the lane, and the pointers are marked as global memory: the loads and stores then take the
// "scalar base + vector offset" form and no 64-bit address arithmetic is left on the vector ALU.
typedef const __attribute__((address_space(1))) uint8_t* gcptr_t;
typedef __attribute__((address_space(1))) uint8_t* gptr_t;

// A pointer marked as global memory, for the accesses that are not of that form (ragged ends, a group's scale): of a
// pointer that comes from the tensor table the compiler does not know what it points to, and a single FLAT access in a
// kernel makes it wait for every outstanding load wherever the paths join, the one without the access included.
template <typename T>
__device__ __forceinline__ __attribute__((address_space(1))) T* as_global(T* p) {
    return (__attribute__((address_space(1))) T*)p;
}

// The base is passed through readfirstlane (a register copy for a value that is already uniform)
// so that the compiler keeps it apart from the lane offset instead of folding both into one
// 64-bit vector address.
__device__ __forceinline__ uint64_t uniform_u64(uint64_t v) {
    const uint32_t lo = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)v);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(v >> 32));
    return ((uint64_t)hi << 32) | lo;
}
__device__ __forceinline__ gcptr_t gbase(const void* p, int64_t byte_off) {
    return (gcptr_t)uniform_u64((uint64_t)p + (uint64_t)byte_off);
}
__device__ __forceinline__ gptr_t gbase(void* p, int64_t byte_off) {
    return (gptr_t)uniform_u64((uint64_t)p + (uint64_t)byte_off);
}

// Redefines a 32-bit lane offset at the point of use (an empty asm statement, no instruction):
// its zero-extension then stays next to the access it feeds, which the "scalar base + 32-bit
// vector offset" addressing form requires.
__device__ __forceinline__ uint32_t block_local(uint32_t v) {
    asm volatile("" : "+v"(v));
    return v;
}

// Element i of packed BF16 values, as FP32.
template <int N>
__device__ __forceinline__ float bf16_of(const uint32_t (&w)[N], int i) {
    return (i & 1) ? u2f(w[i >> 1] & 0xffff0000u) : u2f(w[i >> 1] << 16);
}

// Stores of the streaming data are non-temporal, and where THROUGH at device scope (sc1) on top of that: a line then goes on
// to memory as it is written, instead of when the L2 needs its place or the kernel ends.  The launches say which (see
// step_through).  Only the buffer instructions let a program choose (aux: bit 1 nt, bit 4 sc1); the descriptor holds the
// base, no upper bound (the callers' lanes are known to exist) and 32-bit raw data.
constexpr int kNonTemporalThrough = 2 | 16;
__device__ __forceinline__ __amdgpu_buffer_rsrc_t store_rsrc(gptr_t base) {
    return __builtin_amdgcn_make_buffer_rsrc((void*)base, 0, -1, 0x00027000);
}

// 4 * N bytes from / to base + byte_off (4N-byte aligned, N <= 4)
template <int N>
__device__ __forceinline__ void gld(uint32_t (&w)[N], gcptr_t base, uint32_t byte_off) {
    static_assert(N == 1 || N == 2 || N == 4, "");
    typedef uint32_t vec_t __attribute__((ext_vector_type(N)));
    typedef const __attribute__((address_space(1))) vec_t* vptr_t;
    const vec_t v = __builtin_nontemporal_load((vptr_t)(base + byte_off));
#pragma unroll
    for (int k = 0; k < N; ++k) w[k] = v[k];
}
template <bool THROUGH, int N>
__device__ __forceinline__ void gst(gptr_t base, uint32_t byte_off, const uint32_t (&w)[N]) {
    static_assert(N == 1 || N == 2 || N == 4, "");
    typedef uint32_t vec_t __attribute__((ext_vector_type(N)));
    typedef __attribute__((address_space(1))) vec_t* vptr_t;
    vec_t v;
#pragma unroll
    for (int k = 0; k < N; ++k) v[k] = w[k];
    if constexpr (!THROUGH) __builtin_nontemporal_store(v, (vptr_t)(base + byte_off));
    else if constexpr (N == 1) __builtin_amdgcn_raw_buffer_store_b32(w[0], store_rsrc(base), byte_off, 0, kNonTemporalThrough);
    else if constexpr (N == 2) __builtin_amdgcn_raw_buffer_store_b64(v, store_rsrc(base), byte_off, 0, kNonTemporalThrough);
    else __builtin_amdgcn_raw_buffer_store_b128(v, store_rsrc(base), byte_off, 0, kNonTemporalThrough);
}
// 4 * N bytes as consecutive 16-byte (or one 8-byte) accesses
template <int N>
__device__ __forceinline__ void gld_words(uint32_t (&w)[N], gcptr_t base, uint32_t byte_off) {
    if constexpr (N <= 4) {
        gld(w, base, byte_off);
    } else {
        static_assert(N % 4 == 0, "");
#pragma unroll
        for (int k = 0; k < N / 4; ++k) {
            uint32_t t[4];
            gld(t, base, byte_off + 16u * k);
            w[4 * k] = t[0]; w[4 * k + 1] = t[1]; w[4 * k + 2] = t[2]; w[4 * k + 3] = t[3];
        }
    }
}
template <bool THROUGH, int N>
__device__ __forceinline__ void gst_words(gptr_t base, uint32_t byte_off, const uint32_t (&w)[N]) {
    if constexpr (N <= 4) {
        gst<THROUGH>(base, byte_off, w);
    } else {
        static_assert(N % 4 == 0, "");
#pragma unroll
        for (int k = 0; k < N / 4; ++k) {
            const uint32_t t[4] = {w[4 * k], w[4 * k + 1], w[4 * k + 2], w[4 * k + 3]};
            gst<THROUGH>(base, byte_off + 16u * k, t);
        }
    }
}
// FP32 streams: four floats per lane, so that one access of a wavefront covers 1 KB of consecutive bytes.
typedef float f32x4_t __attribute__((ext_vector_type(4)));
__device__ __forceinline__ void gld_floats(float (&f)[4], gcptr_t base, uint32_t byte_off) {
    const f32x4_t v = __builtin_nontemporal_load((const __attribute__((address_space(1))) f32x4_t*)(base + byte_off));
    f[0] = v[0]; f[1] = v[1]; f[2] = v[2]; f[3] = v[3];
}
template <bool THROUGH>
__device__ __forceinline__ void gst_floats(gptr_t base, uint32_t byte_off, const float (&f)[4]) {
    const uint32_t w[4] = {f2u(f[0]), f2u(f[1]), f2u(f[2]), f2u(f[3])};
    gst<THROUGH>(base, byte_off, w);
}
__device__ __forceinline__ uint32_t gld_u16(gcptr_t base, uint32_t byte_off) {
    return *(const __attribute__((address_space(1))) uint16_t*)(base + byte_off);
}
__device__ __forceinline__ void gst_u16(gptr_t base, uint32_t byte_off, uint32_t v) {
    *(__attribute__((address_space(1))) uint16_t*)(base + byte_off) = (uint16_t)v;
}

// A full lane: tile0 = index of the tile's first element in the tensor (wave-uniform, a multiple
// of 32), lane_el = index of the lane's first element inside the tile (a multiple of VEC).
template <int VEC, bool HAS_V, bool SPLIT, bool QUANT>
__device__ __forceinline__ void load_full(LaneIO<VEC>& x, const TensorDev& T, int64_t tile0, uint32_t lane_el) {
    lane_el = block_local(lane_el);
    if constexpr (SPLIT) {
        gld_words(x.p, gbase(T.param, 2 * tile0), 2u * lane_el);
        gld_words(x.r, gbase(T.rho, tile0), lane_el);
    } else {
        gld_floats(x.th32, gbase(T.theta32, 4 * tile0), 4u * lane_el);
    }
    gld_words(x.g, gbase(T.grad, 2 * tile0), 2u * lane_el);
    if constexpr (QUANT) {
        const uint32_t scale_off = (lane_el >> 5) * 2u;
        gld_words(x.mq, gbase(T.m_q, tile0), lane_el);
        x.ms = gld_u16(gbase(T.m_scale, (tile0 >> 5) * 2), scale_off);
        if (HAS_V) {
            gld_words(x.vq, gbase(T.v_q, tile0), lane_el);
            x.vs = gld_u16(gbase(T.v_scale, (tile0 >> 5) * 2), scale_off);
        }
    } else {
        gld_floats(x.m32, gbase(T.m32, 4 * tile0), 4u * lane_el);
        if constexpr (HAS_V) gld_floats(x.v32, gbase(T.v32, 4 * tile0), 4u * lane_el);
    }
}

// Ragged end of a tensor: the cnt < VEC elements that a lane still has, one by one, missing elements as zero (a zero
// element yields zero moments and therefore never raises its group's absmax).  Every load is issued, those of missing
// elements from the last existing one, so that all of a lane's loads are in flight together: written as "load it if it
// exists", each became a branch with a wait behind its load, and the list of 25 small odd sizes spent most of its
// kernel time in this chain of about 40 loads.  cnt >= 1: a lane without elements has no last one, its caller reads nothing.
template <int N, typename T>
__device__ __forceinline__ void load_elements(T (&e)[N], const T* elements, int cnt) {
    const auto p = as_global(elements);
#pragma unroll
    for (int i = 0; i < N; ++i) e[i] = p[i < cnt ? i : cnt - 1];
#pragma unroll
    for (int i = 0; i < N; ++i) if (i >= cnt) e[i] = (T)0;
}
template <int N>
__device__ __forceinline__ void pack_elements(uint32_t (&w)[N / 4], const uint8_t (&e)[N]) {
#pragma unroll
    for (int j = 0; j < N / 4; ++j)
        w[j] = (uint32_t)e[4 * j] | ((uint32_t)e[4 * j + 1] << 8) | ((uint32_t)e[4 * j + 2] << 16) |
               ((uint32_t)e[4 * j + 3] << 24);
}
template <int N>
__device__ __forceinline__ void pack_elements(uint32_t (&w)[N / 2], const uint16_t (&e)[N]) {
#pragma unroll
    for (int j = 0; j < N / 2; ++j) w[j] = (uint32_t)e[2 * j] | ((uint32_t)e[2 * j + 1] << 16);
}

// Missing weights are 1, so that SGD and Lion wavefronts that have some keep to the short forms of Algorithm 1.  (In AdamW the
// root of a missing element's variance, 0, is NaN on the short path, and so is its new weight: the wavefront takes the general
// form of the split, with the same bits.)
template <int VEC, bool HAS_V, bool SPLIT, bool QUANT>
__device__ __forceinline__ void load_tail(LaneIO<VEC>& x, const TensorDev& T, int64_t off, int cnt) {
    x = LaneIO<VEC>{};
    if constexpr (SPLIT) {
#pragma unroll
        for (int j = 0; j < VEC / 2; ++j) x.p[j] = 0x3f803f80u;
    }
    if (cnt == 0) return;
    uint16_t g[VEC], p[VEC];
    uint8_t r[VEC], mq[VEC], vq[VEC];
    load_elements(g, reinterpret_cast<const uint16_t*>(T.grad) + off, cnt);
    if constexpr (SPLIT) {
        load_elements(p, reinterpret_cast<const uint16_t*>(T.param) + off, cnt);
        load_elements(r, reinterpret_cast<const uint8_t*>(T.rho) + off, cnt);
    } else {
        load_elements(x.th32, T.theta32 + off, cnt);
    }
    if constexpr (QUANT) {
        load_elements(mq, reinterpret_cast<const uint8_t*>(T.m_q) + off, cnt);
        x.ms = as_global(T.m_scale)[off >> 5];
        if constexpr (HAS_V) {
            load_elements(vq, T.v_q + off, cnt);
            x.vs = as_global(T.v_scale)[off >> 5];
        }
    } else {
        load_elements(x.m32, T.m32 + off, cnt);
        if constexpr (HAS_V) load_elements(x.v32, T.v32 + off, cnt);
    }
    pack_elements(x.g, g);
    if constexpr (SPLIT) {
#pragma unroll
        for (int i = 0; i < VEC; ++i) if (i >= cnt) p[i] = 0x3f80u;
        pack_elements(x.p, p);
        pack_elements(x.r, r);
    }
    if constexpr (QUANT) {
        pack_elements(x.mq, mq);
        if constexpr (HAS_V) pack_elements(x.vq, vq);
    }
}

template <int VEC, bool HAS_V, bool SPLIT, bool QUANT, bool THROUGH>
__device__ __forceinline__ void store_full(const LaneIO<VEC>& y, const TensorDev& T, int64_t tile0, uint32_t lane_el,
                                           bool group_leader) {
    lane_el = block_local(lane_el);
    if constexpr (SPLIT) {
        gst_words<THROUGH>(gbase(T.param, 2 * tile0), 2u * lane_el, y.p);
        gst_words<THROUGH>(gbase(T.rho, tile0), lane_el, y.r);
    } else {
        gst_floats<THROUGH>(gbase(T.theta32, 4 * tile0), 4u * lane_el, y.th32);
    }
    if constexpr (QUANT) {
        gst_words<THROUGH>(gbase(T.m_q, tile0), lane_el, y.mq);
        if (HAS_V) gst_words<THROUGH>(gbase(T.v_q, tile0), lane_el, y.vq);
        if (group_leader) {
            const uint32_t scale_off = (lane_el >> 5) * 2u;
            gst_u16(gbase(T.m_scale, (tile0 >> 5) * 2), scale_off, y.ms);
            if (HAS_V) gst_u16(gbase(T.v_scale, (tile0 >> 5) * 2), scale_off, y.vs);
        }
    } else {
        gst_floats<THROUGH>(gbase(T.m32, 4 * tile0), 4u * lane_el, y.m32);
        if constexpr (HAS_V) gst_floats<THROUGH>(gbase(T.v32, 4 * tile0), 4u * lane_el, y.v32);
    }
}

template <int VEC, bool HAS_V, bool SPLIT, bool QUANT>
__device__ __forceinline__ void store_tail(const LaneIO<VEC>& y, const TensorDev& T, int64_t off, int cnt,
                                           bool group_leader) {
    const auto p = as_global(reinterpret_cast<uint16_t*>(T.param)) + off;
    const auto r = as_global(reinterpret_cast<uint8_t*>(T.rho)) + off;
    const auto mq = as_global(reinterpret_cast<uint8_t*>(T.m_q)) + off;
    const auto vq = as_global(T.v_q) + off;
#pragma unroll
    for (int i = 0; i < VEC; ++i) {
        if (i < cnt) {
            if (SPLIT) {
                p[i] = (uint16_t)(y.p[i >> 1] >> (16 * (i & 1)));
                r[i] = (uint8_t)(y.r[i >> 2] >> (8 * (i & 3)));
            } else {
                as_global(T.theta32)[off + i] = y.th32[i];
            }
            if (QUANT) {
                mq[i] = (uint8_t)(y.mq[i >> 2] >> (8 * (i & 3)));
                if (HAS_V) vq[i] = (uint8_t)(y.vq[i >> 2] >> (8 * (i & 3)));
            } else {
                as_global(T.m32)[off + i] = y.m32[i];
                if (HAS_V) as_global(T.v32)[off + i] = y.v32[i];
            }
        }
    }
    if (QUANT && group_leader && cnt > 0) {
        as_global(T.m_scale)[off >> 5] = (uint16_t)y.ms;
        if (HAS_V) as_global(T.v_scale)[off >> 5] = (uint16_t)y.vs;
    }
}

// ------------------------------------------------------- the per-lane update --
//
// Splits (or stores as FP32) the new master weights of a lane.
template <int VEC, bool SPLIT>
__device__ __forceinline__ void split_lane(LaneIO<VEC>& y, const float (&tht)[VEC]) {
    if constexpr (SPLIT) {
        float lowest = 3.0e38f;
#pragma unroll
        for (int i = 0; i < VEC; ++i) lowest = min_or_nan(lowest, fabsf(tht[i]));
#pragma unroll
        for (int j = 0; j < VEC / 2; ++j) y.p[j] = bf16_pack(tht[2 * j], tht[2 * j + 1]);
        uint32_t c[VEC];
        if (!any_lane(!(lowest >= kSplitFastLo))) {
#pragma unroll
            for (int i = 0; i < VEC; ++i) c[i] = rho_bits_fast(tht[i], bf16_of(y.p, i));
        } else {
#pragma unroll
            for (int i = 0; i < VEC; ++i) c[i] = rho_bits_general(tht[i], bf16_of(y.p, i));
        }
#pragma unroll
        for (int j = 0; j < VEC / 4; ++j) y.r[j] = pack_low_bytes(c[4 * j], c[4 * j + 1], c[4 * j + 2], c[4 * j + 3]);
    } else {
#pragma unroll
        for (int i = 0; i < VEC; ++i) y.th32[i] = tht[i];
    }
}

// The master weights of a lane.
template <int VEC, bool SPLIT>
__device__ __forceinline__ void master_weights(const LaneIO<VEC>& x, const StepTables& tab, float (&th)[VEC]) {
    if constexpr (SPLIT) {
        float q[VEC], lowest = 3.0e38f;
#pragma unroll
        for (int i = 0; i < VEC; ++i) {
            q[i] = tab.rho_scaled[(x.r[i >> 2] >> (8 * (i & 3))) & 0xffu];
            th[i] = reconstruct_fast(bf16_of(x.p, i), q[i]);
            lowest = min_or_nan(lowest, fabsf(th[i]));
        }
        if (any_lane(!(lowest >= kSplitFastLo))) {
#pragma unroll
            for (int i = 0; i < VEC; ++i) th[i] = reconstruct_general(bf16_of(x.p, i), q[i]);
        }
    } else {
#pragma unroll
        for (int i = 0; i < VEC; ++i) th[i] = x.th32[i];
    }
}

// KIND: 0 AdamW (Algorithm 4), 1 SGD (Algorithm 5), 2 Lion (Algorithm 6).
// Operates on the VEC elements of one lane; the lanes holding the rest of the same 32-element
// group (the lane's quad when VEC == 8, its run of eight lanes when VEC == 4) must execute this function with it.
// SPLIT / QUANT: the paper's ablations (Section 4.3).  SPLIT = false keeps the master weight in
// FP32 (x.th32 -> y.th32); QUANT = false keeps the states in FP32 (x.m32, x.v32 -> y.m32, y.v32).
// EXACT (AdamW only): the quotient m_hat / (sqrt(v_hat) + eps) is the correctly rounded one for every
// input; otherwise it is the faithful form above.  Everything else, the square root, the state codes and
// the scales included, is exact in both modes.
// M_HAT (AdamW only): the momentum's bias correction is not 1; otherwise (from step 165 on with beta1 = 0.9) m_hat = m_t.
// cnt: the elements of the lane that exist (VEC where FULL).
template <int KIND, int VEC, bool SPLIT, bool QUANT, bool EXACT, bool M_HAT, bool FULL>
__device__ __forceinline__ void update_lane(const LaneIO<VEC>& x, LaneIO<VEC>& y, const StepTables& tab,
                                            const StepConsts& c, float lr, float wd, int cnt) {
    constexpr bool HAS_V = (KIND == 0);
    const float s_m = QUANT ? (float)__builtin_bit_cast(_Float16, (uint16_t)x.ms) : 0.0f;
    const float s_v = (QUANT && HAS_V) ? (float)__builtin_bit_cast(_Float16, (uint16_t)x.vs) : 0.0f;

    float mt[VEC];    // new momentum
    float vt[VEC];    // new variance (AdamW)
    float rh[VEC];    // sqrt of the bias-corrected new variance (AdamW)
    float th[VEC];    // master weights, replaced by the new ones
    float amax_m = 0.0f, amax_v = 0.0f;
    float amin_m = 3.0e38f, amin_v = 3.0e38f;     // AdamW: smallest |m_t| and v_t of the lane
    bool fast = false;                            // AdamW: the wavefront takes the short square root and division

    // prologue: reconstruct master weights and optimizer state
    master_weights<VEC, SPLIT>(x, tab, th);
#pragma unroll
    for (int i = 0; i < VEC; ++i) {
        const float g = bf16_of(x.g, i);
        float m;
        if (QUANT) m = tab.m[(x.mq[i >> 2] >> (8 * (i & 3))) & 0xffu] * s_m;       // Q_m^-1
        else m = x.m32[i];
        float m_new;
        if (KIND == 0) {
            float v;
            if (QUANT) {
                const float v1 = code_over_255((x.vq[i >> 2] >> (8 * (i & 3))) & 0xffu) * s_v;     // Q_v^-1
                v = v1 * v1;
            } else {
                v = x.v32[i];
            }
            m_new = (c.beta1 * m) + (c.omb1 * g);
            const float gg = g * g;
            const float v_new = (c.beta2 * v) + (c.omb2 * gg);
            vt[i] = v_new;
            amax_v = fmaxf(amax_v, v_new);
            if (FULL || i < cnt) {          // (an element that does not exist has zero moments)
                amin_v = fminf(amin_v, v_new);
                amin_m = fminf(amin_m, fabsf(m_new));
            }
        } else if (KIND == 1) {
            m_new = (c.beta1 * m) + g;                           // beta1 carries the momentum mu
            th[i] = th[i] - (lr * (m_new + (wd * th[i])));
        } else {
            const float cc = (c.beta1 * m) + (c.omb1 * g);
            const float u = (cc > 0.0f) ? 1.0f : ((cc < 0.0f) ? -1.0f : 0.0f);
            m_new = (c.beta2 * m) + (c.omb2 * g);
            th[i] = th[i] - (lr * (u + (wd * th[i])));
        }
        mt[i] = m_new;
        amax_m = fmaxf(amax_m, fabsf(m_new));
    }
    if (KIND == 0) {
        // One wave-uniform range test, on the raw extremes of every lane, selects the short square root
        // and the short division for the whole wavefront (else sqrtf and the IEEE division throughout: same
        // results).  The bias corrections rbc1, rbc2 are at least 1 and multiplying by them is monotone, so
        //   v_t >= 2^-96 for every element   =>  v_hat, and v_t itself, are in the short square root's range;
        //   v_t <= c.v_max (2^60 / rbc2, rounded down)   =>  v_hat <= 2^60: finite, and sqrt(v_hat) + eps is a
        //                                                    denominator well inside the normal range;
        //   |m_t| <= c.m_max (2^60 / rbc1, rounded down) and, for the correctly rounded division only,
        //   |m_t| >= 2^-60   =>  the numerator m_hat is in the short division's range.
        // The host sets v_max = m_max = -1 when eps is outside [2^-60, 1], and sqrt_min = +inf when the short
        // square root is not to be used on this device: every test then fails.  Exact zeros fail it too.
        fast = !(any_lane(!(amax_v <= c.v_max)) | any_lane(!(amin_v >= c.sqrt_min)) |
                 any_lane(!(amax_m <= c.m_max)) | (EXACT ? any_lane(!(amin_m >= kDivFastLo)) : false));
#pragma unroll
        for (int j = 0; j < VEC / 4; ++j) {
            float mh4[4], vh4[4], quo[4];
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                mh4[k] = M_HAT ? mt[4 * j + k] * c.rbc1 : mt[4 * j + k];
                vh4[k] = vt[4 * j + k] * c.rbc2;
            }
            if (!fast) {
#pragma unroll
                for (int k = 0; k < 4; ++k) rh[4 * j + k] = sqrtf(vh4[k]);
            } else {
#pragma unroll
                for (int k = 0; k < 4; ++k) rh[4 * j + k] = sqrt_rn_midrange(vh4[k]);
            }
            if (!fast) {
#pragma unroll
                for (int k = 0; k < 4; ++k) quo[k] = mh4[k] / (rh[4 * j + k] + c.eps);
            } else if (EXACT) {
#pragma unroll
                for (int k = 0; k < 4; ++k) quo[k] = div_rn_midrange(mh4[k], rh[4 * j + k] + c.eps);
            } else {
#pragma unroll
                for (int k = 0; k < 4; ++k) quo[k] = div_faithful(mh4[k], rh[4 * j + k] + c.eps);
            }
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const float upd = quo[k] + (wd * th[4 * j + k]);
                th[4 * j + k] = th[4 * j + k] - (lr * upd);
            }
        }
    }
    // epilogue, part 1: split the new master weights
    split_lane<VEC, SPLIT>(y, th);
    if (!QUANT) {
#pragma unroll
        for (int i = 0; i < VEC; ++i) {
            y.m32[i] = mt[i];
            if (HAS_V) y.v32[i] = vt[i];
        }
        return;
    }

    // epilogue, part 2: group scales (DPP steps join the lanes of a group).  The square root
    // is monotone, so the group maximum of sqrt(v) is the square root of the maximum of v.
    amax_m = group_max<VEC>(amax_m);
    float s_m_new, s_v_new, r_v = 0.0f, kr255 = 0.0f;
    y.ms = group_scale(amax_m, &s_m_new);
    const float r_m = recip_of_scale(s_m_new);
    if (HAS_V) {
        // the group's maximum lies between the extremes of the wavefront's lanes: in the short root's range if they are
        amax_v = group_max<VEC>(amax_v);
        const float root_max = fast ? sqrt_rn_midrange(amax_v) : sqrtf(amax_v);
        y.vs = group_scale(root_max, &s_v_new);
        r_v = recip_of_scale(s_v_new);
        // 255 * sqrt(1 / rbc2) * r_v to within one rounding: the constant comes from the host as the two halves of
        // its double-precision value
        kr255 = fmaf(c.k255_hi, r_v, c.k255_lo * r_v);
    }
    const bool vt_root_general = !fast;
    // epilogue: state codes, four at a time (one word of each code stream).  Each code is converted
    // twice, from the two ends of an interval that contains the exact argument of Round(); where the
    // two words differ some element of the block may sit on the other side of a rounding tie, and the
    // block is recomputed with the exact sequence (for the whole wavefront: a few percent of the blocks).
#pragma unroll
    for (int j = 0; j < VEC / 4; ++j) {
        uint32_t lo_w = 0, hi_w = 0;
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            float lo, hi;
            m_code_bracket(mt[4 * j + k], r_m, &lo, &hi);
            lo_w = put_u8(lo, k, lo_w);
            hi_w = put_u8(hi, k, hi_w);
        }
        if (any_lane(lo_w != hi_w)) {
            y.mq[j] = pack_low_bytes(m_code_exact(mt[4 * j], r_m), m_code_exact(mt[4 * j + 1], r_m),
                                     m_code_exact(mt[4 * j + 2], r_m), m_code_exact(mt[4 * j + 3], r_m));
        } else {
            y.mq[j] = lo_w ^ 0x80808080u;      // code + 128 -> two's complement
        }
        if (HAS_V) {
            lo_w = 0; hi_w = 0;
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                float lo, hi;
                v_code_bracket(rh[4 * j + k], kr255, &lo, &hi);
                lo_w = put_u8(lo, k, lo_w);
                hi_w = put_u8(hi, k, hi_w);
            }
            if (any_lane(lo_w != hi_w)) {
                // exact recomputation; the short exact root serves when every v_t of the wavefront
                // is in its range (v_t and v_hat differ by the factor rbc2 >= 1: a separate test)
                uint32_t cv[4];
                if (vt_root_general) {
#pragma unroll
                    for (int k = 0; k < 4; ++k) cv[k] = v_code_exact(vt[4 * j + k], r_v);
                } else {
#pragma unroll
                    for (int k = 0; k < 4; ++k) cv[k] = v_code_exact_midrange(vt[4 * j + k], r_v);
                }
                y.vq[j] = pack_low_bytes(cv[0], cv[1], cv[2], cv[3]);
            } else {
                y.vq[j] = lo_w;
            }
        }
    }
}

// ------------------------------------------------------------ step kernels --
// The tensor that holds workgroup b of a list.  Every load is wave-uniform (scalar).
__device__ __forceinline__ uint32_t locate_tensor(const TensorDev* tensors, const uint32_t* coarse, uint32_t shift, uint32_t b) {
    const uint32_t* entry = coarse + (b >> shift);
    const uint32_t t = entry[0];
    return shift ? entry_of(b, t, entry[1], [&](uint32_t i) { return tensors[i].first_tile; }) : t;
}
// The tensor and the tile within it that workgroup blockIdx.x handles.
template <bool DIRECT>
__device__ __forceinline__ int64_t locate_tile(const StepArgs& a, TensorDev& T) {
    const uint32_t b = blockIdx.x + a.block_offset;
    if (DIRECT) {
        T = a.single;
        return (int64_t)b;
    }
    T = a.tensors[locate_tensor(a.tensors, a.coarse, a.coarse_shift, b)];
    return (int64_t)(b - T.first_tile);
}

// What a step's kernels take.  The first arguments are those that its streaming loads wait for, fourteen words that the command
// processor has in registers before a wavefront starts; the others come by loads of their own, which the kernels wait for behind the
// streaming loads.  Only what a kind reads is passed (a byte costs the host 2.6 ns).  With one struct of 200 bytes for all, launched by
// <<<>>>, -> without -> with preloaded arguments, us a call: AdamW over 2^20 elements 4.72 -> 4.71 -> 4.56, 2^21 6.30 -> 6.28 -> 6.12, 25 odd sizes
// 4.33 -> 4.10 -> 4.05; SGD 2^21 4.26 -> 4.23 -> 4.05, 2^22 6.21 -> 6.34 -> 5.95, ten tensors of 5 M 9.37 -> 9.29 -> 9.06, ResNet-50 40.9 -> 40.8 -> 40.5.
// (Where the host sets the pace, its differ more from run to run than this: AdamW over 2^20 elements on another machine 5.07 -> 5.01.  The kernel alone
// takes 4.6 there, 5.0 before.)
template <bool DIRECT, bool HAS_V>
struct TensorArgs {};       // (of a list: everything is in the table)
template <>
struct TensorArgs<true, false> {
    uint16_t* m_scale;
    float lr, wd;
    explicit TensorArgs(const TensorDev& d) : m_scale(d.m_scale), lr(d.lr), wd(d.wd) {}
};
template <>
struct TensorArgs<true, true> : TensorArgs<true, false> {
    uint16_t* v_scale;
    explicit TensorArgs(const TensorDev& d) : TensorArgs<true, false>(d), v_scale(d.v_scale) {}
};
template <bool HAS_V>
struct TensorArgs<false, HAS_V> {
    explicit TensorArgs(const TensorDev&) {}
};
template <int KIND>
struct KindConsts;
template <>
struct KindConsts<0> {
    const float* sqrt_min_word;
    float beta1, beta2, omb1, omb2, rbc1, rbc2, eps, k255_hi, k255_lo, v_max, m_max;
    explicit KindConsts(const StepArgs& a)
        : sqrt_min_word(a.sqrt_min_word), beta1(a.c.beta1), beta2(a.c.beta2), omb1(a.c.omb1), omb2(a.c.omb2), rbc1(a.c.rbc1),
          rbc2(a.c.rbc2), eps(a.c.eps), k255_hi(a.c.k255_hi), k255_lo(a.c.k255_lo), v_max(a.c.v_max), m_max(a.c.m_max) {}
    // sqrt_min is one more scalar load.  The word counts as constant: the check that writes it may run beside a step on another
    // stream, but only once per device, and the results are the same with either value.
    __device__ __forceinline__ StepConsts get() const {
        return {beta1, beta2, omb1, omb2, rbc1, rbc2, eps, k255_hi, k255_lo, v_max, m_max,
                *(const __attribute__((address_space(4))) float*)sqrt_min_word};
    }
};
template <>
struct KindConsts<1> {
    float momentum;
    explicit KindConsts(const StepArgs& a) : momentum(a.c.beta1) {}
    __device__ __forceinline__ StepConsts get() const { return {momentum}; }
};
template <>
struct KindConsts<2> {
    float beta1, beta2, omb1, omb2;
    explicit KindConsts(const StepArgs& a) : beta1(a.c.beta1), beta2(a.c.beta2), omb1(a.c.omb1), omb2(a.c.omb2) {}
    __device__ __forceinline__ StepConsts get() const { return {beta1, beta2, omb1, omb2}; }
};
// The kernel is overloaded by the type of its last argument, one overload for each way of doing the same step: AdamW with and
// without a bias correction of the momentum that is not 1 (an instruction per element less is 0.3-0.9 % of a step's time:
// GPT-2 253.0 -> 251.9 us, Llama layer 445.6 -> 441.9), and either kind of stores (a branch in the kernel instead costs plain
// FP32 steps over a few million elements 1 %).
template <int KIND, bool DIRECT, bool M_HAT, bool THROUGH>
struct VariantArgs : TensorArgs<DIRECT, KIND == 0>, KindConsts<KIND> {
    explicit VariantArgs(const StepArgs& a) : TensorArgs<DIRECT, KIND == 0>(a.single), KindConsts<KIND>(a) {}
};
// The first arguments.  Of one tensor, the arrays that the variant has, the element count (low half, high half) and the first
// workgroup's tile; of a list, p0 the table, p1 the coarse table, u0 its shift, u1 and u3 what makes the rate (StepArgs).
struct HotArgs {
    const void *p0, *p1, *p2, *p3, *p4;
    uint32_t u0, u1, block_offset, u3;
};
template <bool DIRECT, bool SPLIT, bool QUANT>
static HotArgs hot_args(const StepArgs& a) {
    const TensorDev& d = a.single;
    if (!DIRECT) return {a.tensors, a.coarse, nullptr, nullptr, nullptr, a.coarse_shift, a.table_lr_mask, a.block_offset, a.shared_lr_bits};
    return {SPLIT ? d.param : (const void*)d.theta32, SPLIT ? d.rho : nullptr, d.grad, QUANT ? d.m_q : (const void*)d.m32,
            QUANT ? d.v_q : (const void*)d.v32, (uint32_t)d.numel, (uint32_t)((uint64_t)d.numel >> 32), a.block_offset, 0};
}

// First element, in its tensor, of what this wavefront handles of a workgroup of WAVES with tile `tile`, where the tiles of whole
// groups are dealt out (wave_part).  Wave-uniform.  (Copies: bytes of a segment.)
template <int WAVES, int WAVE_ELEMS>
__device__ __forceinline__ int64_t wave_start(int64_t tile, int64_t numel) {
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    return wave_part(tile, wave, WAVES, numel / (WAVES * WAVE_ELEMS)) * WAVE_ELEMS;
}

// The elements from tile0 on, `rem` of them in the tensor; lane_el is the first one of the lane, counted from there.
// FULL: every lane of the workgroup holds VEC elements (all tiles of a
// tensor but possibly its last); the code then has no per-lane case distinction at all.
// (Variants in which a workgroup loads two or four such tiles up front and then updates them in
// turn - fewer look-ups, more bytes in flight per workgroup - ran at the same rate.)
template <int KIND, int VEC, int THREADS, bool SPLIT, bool QUANT, bool EXACT, bool M_HAT, bool THROUGH, bool FULL>
__device__ __forceinline__ void step_tile(const TensorDev& T, const KindConsts<KIND>& consts, StepTables& tab,
                                          const TableEntries& entries, int64_t tile0, uint32_t lane_el, int rem, int tid) {
    constexpr bool HAS_V = (KIND == 0);
    const bool leader = (tid & (kGroup / VEC - 1)) == 0;
    // the number of them that fall to this lane
    const int left = rem - (int)lane_el;
    const int cnt = FULL ? VEC : (left >= VEC ? VEC : (left > 0 ? left : 0));
    LaneIO<VEC> x, y;
    if (FULL || cnt == VEC) load_full<VEC, HAS_V, SPLIT, QUANT>(x, T, tile0, lane_el);
    else load_tail<VEC, HAS_V, SPLIT, QUANT>(x, T, tile0 + lane_el, cnt);
    if constexpr (SPLIT || QUANT) {        // the plain FP32 step decodes nothing
        store_table_entries<THREADS, SPLIT, QUANT>(tab, entries, tid);
        __syncthreads();
    }
    const StepConsts c = consts.get();       // (behind the streaming loads)
    // All lanes of a group run the update together (a lane with cnt == 0 may share its group
    // with lanes that hold elements); lanes past the end compute on zeros and store nothing.
    update_lane<KIND, VEC, SPLIT, QUANT, EXACT, M_HAT, FULL>(x, y, tab, c, T.lr, T.wd, cnt);
    if (FULL || cnt == VEC) store_full<VEC, HAS_V, SPLIT, QUANT, THROUGH>(y, T, tile0, lane_el, leader);
    else store_tail<VEC, HAS_V, SPLIT, QUANT>(y, T, tile0 + lane_el, cnt, leader);
}

// A workgroup handles one tile of one tensor and then retires (persistent workgroups that loop
// over many tiles were measured 10 % slower: an iteration's loads then wait behind the previous
// iteration's stores).  Order of issue: decode-table loads, the (tensor, tile) look-up, the
// streaming loads; then the tables go to LDS.
template <int KIND, int VEC, int THREADS, bool DIRECT, bool SPLIT, bool QUANT, bool EXACT, bool M_HAT, bool THROUGH>
__device__ __forceinline__ void step_workgroup(const HotArgs& h, const VariantArgs<KIND, DIRECT, M_HAT, THROUGH>& a) {
    constexpr int kTile = THREADS * VEC;       // elements per workgroup
    __shared__ StepTables tab;
    const int tid = (int)threadIdx.x;
    TableEntries entries;
    if constexpr (SPLIT || QUANT) load_table_entries<THREADS, SPLIT, QUANT>(entries, tid);
    const uint32_t b = blockIdx.x + h.block_offset;
    TensorDev T;
    TensorDev* entry = nullptr;
    if constexpr (DIRECT) {
        T = TensorDev{};
        T.param = T.theta32 = (float*)h.p0;
        T.rho = (int8_t*)h.p1;
        T.grad = h.p2;
        T.m_q = (int8_t*)h.p3;
        T.m32 = (float*)h.p3;
        T.v_q = (uint8_t*)h.p4;
        T.v32 = (float*)h.p4;
        T.numel = (int64_t)((uint64_t)h.u1 << 32 | h.u0);
        T.m_scale = a.m_scale;
        if constexpr (KIND == 0) T.v_scale = a.v_scale;
        T.lr = a.lr;
        T.wd = a.wd;
    } else {
        TensorDev* tensors = (TensorDev*)h.p0;
        entry = tensors + locate_tensor(tensors, (const uint32_t*)h.p1, h.u0, b);
        T = *entry;
    }
    const int64_t chunk = DIRECT ? (int64_t)b : (int64_t)(b - T.first_tile);
    // first element of the tile, or where tiles are dealt out of this wavefront's part of them (wave-uniform)
    constexpr bool DEALT = step_dealt(KIND, SPLIT, QUANT, THROUGH);
    const int64_t tile0 = DEALT ? wave_start<THREADS / 64, 64 * VEC>(chunk, T.numel) : chunk * (int64_t)kTile;
    const uint32_t lane_el = (uint32_t)(DEALT ? tid & 63 : tid) * VEC;
    const int64_t rem = T.numel - chunk * (int64_t)kTile;      // elements from the tile's first one to the tensor's end
    const float table_lr = T.lr;
    if (!DIRECT) T.lr = u2f((f2u(table_lr) & h.u1) | h.u3);    // (integers: stays on the scalar unit)
    if (rem >= kTile) {
        step_tile<KIND, VEC, THREADS, SPLIT, QUANT, EXACT, M_HAT, THROUGH, true>(T, a, tab, entries, tile0, lane_el, kTile, tid);
    } else {
        // (less than a tile, so within an int; negative for a wavefront behind the tensor's end)
        step_tile<KIND, VEC, THREADS, SPLIT, QUANT, EXACT, M_HAT, THROUGH, false>(T, a, tab, entries, tile0, lane_el,
                                                                                  (int)(T.numel - tile0), tid);
    }
    // (only with a mask of 0: no workgroup of this launch uses what the others read of the entry's rate)
    if (!DIRECT && chunk == 0 && f2u(T.lr) != f2u(table_lr) && tid == 0) entry->lr = T.lr;
}

#define FO_STEP_KERNEL(M_HAT, THROUGH)                                                                                      \
    template <int KIND, int VEC, int THREADS, bool DIRECT, bool SPLIT, bool QUANT, bool EXACT>                              \
    __global__ __launch_bounds__(THREADS) void step_kernel(const void* p0, const void* p1, const void* p2, const void* p3,  \
                                                           const void* p4, uint32_t u0, uint32_t u1, uint32_t block_offset, \
                                                           uint32_t u3, VariantArgs<KIND, DIRECT, M_HAT, THROUGH> a) {      \
        const HotArgs h = {p0, p1, p2, p3, p4, u0, u1, block_offset, u3};                                                   \
        step_workgroup<KIND, VEC, THREADS, DIRECT, SPLIT, QUANT, EXACT, M_HAT, THROUGH>(h, a);                              \
    }
FO_STEP_KERNEL(true, true)
FO_STEP_KERNEL(true, false)
FO_STEP_KERNEL(false, true)
FO_STEP_KERNEL(false, false)
#undef FO_STEP_KERNEL

template <int KIND, bool SPLIT, bool QUANT, bool EXACT, StepShape SHAPE, bool M_HAT, bool THROUGH, bool DIRECT>
static hipError_t launch_direct(const StepArgs& a, unsigned n_blocks, unsigned lds, hipStream_t s) {
    constexpr int VEC = step_vec(SPLIT, QUANT, SHAPE), THREADS = step_threads(SPLIT, QUANT, SHAPE);
    typedef VariantArgs<KIND, DIRECT, M_HAT, THROUGH> args_t;
    void (*kernel)(const void*, const void*, const void*, const void*, const void*, uint32_t, uint32_t, uint32_t, uint32_t, args_t) =
        step_kernel<KIND, VEC, THREADS, DIRECT, SPLIT, QUANT, EXACT>;
    const HotArgs h = hot_args<DIRECT, SPLIT, QUANT>(a);
    return launch(kernel, n_blocks, THREADS, lds, s, h.p0, h.p1, h.p2, h.p3, h.p4, h.u0, h.u1, h.block_offset, h.u3, args_t(a));
}
template <int KIND, bool SPLIT, bool QUANT, bool EXACT, StepShape SHAPE, bool M_HAT, bool THROUGH>
static hipError_t launch_through(bool direct, const StepArgs& a, int64_t n_blocks, hipStream_t s) {
    const int resident = step_resident(KIND, SPLIT, QUANT, SHAPE, direct, n_blocks * chunk_elems(SPLIT, QUANT, SHAPE), THROUGH);
    const unsigned lds = lds_to_hold(resident, SPLIT || QUANT ? sizeof(StepTables) : 0);
    return direct ? launch_direct<KIND, SPLIT, QUANT, EXACT, SHAPE, M_HAT, THROUGH, true>(a, (unsigned)n_blocks, lds, s)
                  : launch_direct<KIND, SPLIT, QUANT, EXACT, SHAPE, M_HAT, THROUGH, false>(a, (unsigned)n_blocks, lds, s);
}
template <int KIND, bool SPLIT, bool QUANT, bool EXACT, StepShape SHAPE, bool M_HAT>
static hipError_t launch_m_hat(bool direct, const StepArgs& a, int64_t n_blocks, hipStream_t s) {
    if constexpr (SHAPE != StepShape::kSmall) {
        if (a.through) return launch_through<KIND, SPLIT, QUANT, EXACT, SHAPE, M_HAT, true>(direct, a, n_blocks, s);
    }
    return launch_through<KIND, SPLIT, QUANT, EXACT, SHAPE, M_HAT, false>(direct, a, n_blocks, s);
}
template <int KIND, bool SPLIT, bool QUANT, bool EXACT, StepShape SHAPE>
static hipError_t launch_variant(bool direct, const StepArgs& a, int64_t n_blocks, hipStream_t s) {
    if constexpr (KIND == 0) {
        if (a.c.rbc1 != 1.0f) return launch_m_hat<KIND, SPLIT, QUANT, EXACT, SHAPE, true>(direct, a, n_blocks, s);
    }
    return launch_m_hat<KIND, SPLIT, QUANT, EXACT, SHAPE, false>(direct, a, n_blocks, s);
}

template <int KIND, bool EXACT>
static hipError_t launch_packed(bool direct, StepShape shape, const StepArgs& a, int64_t n_blocks, hipStream_t s) {
    if (shape == StepShape::kSmall) return launch_variant<KIND, true, true, EXACT, StepShape::kSmall>(direct, a, n_blocks, s);
    if constexpr (KIND != 0) {
        if (shape == StepShape::kWide) return launch_variant<KIND, true, true, EXACT, StepShape::kWide>(direct, a, n_blocks, s);
    }
    return launch_variant<KIND, true, true, EXACT, StepShape::kUsual>(direct, a, n_blocks, s);
}

template <int KIND>
static hipError_t launch_kind(bool direct, bool split, bool quant, StepShape shape, const StepArgs& a, int64_t n_blocks,
                              hipStream_t s) {
    if (split && quant) return launch_packed<KIND, true>(direct, shape, a, n_blocks, s);
    if (split) return launch_variant<KIND, true, false, true, StepShape::kUsual>(direct, a, n_blocks, s);
    if (quant) return launch_variant<KIND, false, true, true, StepShape::kUsual>(direct, a, n_blocks, s);
    return launch_variant<KIND, false, false, true, StepShape::kUsual>(direct, a, n_blocks, s);
}

// exact = false selects the faithful division; it exists for AdamW in the compressed
// layout only (SGD and Lion have neither operation; the ablation variants are always exact).
hipError_t launch_step(int kind, bool direct, bool split, bool quant, StepShape shape, bool exact, const StepArgs& a,
                       int64_t n_blocks, hipStream_t s) {
    if (kind == 0 && !a.sqrt_min_word) return hipErrorInvalidValue;     // the AdamW kernels dereference it
    if (kind == 0 && split && quant && !exact) return launch_packed<0, false>(direct, shape, a, n_blocks, s);
    if (kind == 0) return launch_kind<0>(direct, split, quant, shape, a, n_blocks, s);
    if (kind == 1) return launch_kind<1>(direct, split, quant, shape, a, n_blocks, s);
    return launch_kind<2>(direct, split, quant, shape, a, n_blocks, s);
}

// ------------------------------------------------------------- stream probe --
//
// Moves exactly the bytes of one optimizer step with no arithmetic: every stream the step reads is
// read (gradients included) and every stream it writes is written back unchanged, through the same
// tile look-up, lane layout and access instructions.  Its tiles are dealt out wherever stores go through (wave_part),
// also for AdamW, whose step is faster with them in one piece (step_dealt): for large calls the rate is then the most that the memory
// system was found to give for this traffic, and not what it gives in the step's own order.  (AdamW in one piece -> dealt out, us:
// four Llama layers with embedding and head 3899 -> 3692, 6.4 TB/s, a layer 443 -> 420, GPT-2 243.3 -> 242.8; ResNet-50 51.2 -> 52.5.)
template <int KIND, int VEC, int THREADS, bool DIRECT>
__global__ __launch_bounds__(THREADS) void probe_kernel(StepArgs a) {
    constexpr bool HAS_V = (KIND == 0);
    const int tid = (int)threadIdx.x;
    TensorDev T;
    const int64_t chunk = locate_tile<DIRECT>(a, T);
    const bool leader = (tid & (kGroup / VEC - 1)) == 0;
    const int64_t tile0 = a.through ? wave_start<THREADS / 64, 64 * VEC>(chunk, T.numel) : chunk * (int64_t)(THREADS * VEC);
    const uint32_t lane_el = (uint32_t)(a.through ? tid & 63 : tid) * VEC;
    const int64_t left = T.numel - tile0 - (int64_t)lane_el;
    const int cnt = left >= VEC ? VEC : (left > 0 ? (int)left : 0);
    LaneIO<VEC> x;
    if (cnt == VEC) load_full<VEC, HAS_V, true, true>(x, T, tile0, lane_el);
    else load_tail<VEC, HAS_V, true, true>(x, T, tile0 + lane_el, cnt);
    // The gradient takes no part in what is stored; an empty asm statement that names its registers
    // keeps the load from being removed.
#pragma unroll
    for (int j = 0; j < VEC / 2; ++j) asm volatile("" : : "v"(x.g[j]));
    if (cnt == VEC) {
        if (a.through) store_full<VEC, HAS_V, true, true, true>(x, T, tile0, lane_el, leader);
        else store_full<VEC, HAS_V, true, true, false>(x, T, tile0, lane_el, leader);
    } else store_tail<VEC, HAS_V, true, true>(x, T, tile0 + lane_el, cnt, leader);
}

template <int KIND, StepShape SHAPE>
static hipError_t launch_probe_variant(bool direct, const StepArgs& a, int64_t n_blocks, hipStream_t s) {
    constexpr int VEC = step_vec(true, true, SHAPE), THREADS = step_threads(true, true, SHAPE);
    const dim3 grid((unsigned)n_blocks), block(THREADS);
    const unsigned lds = lds_to_hold(step_resident(KIND, true, true, SHAPE, direct, n_blocks * (THREADS * VEC), a.through), 0);
    if (direct) hipLaunchKernelGGL((probe_kernel<KIND, VEC, THREADS, true>), grid, block, lds, s, a);
    else hipLaunchKernelGGL((probe_kernel<KIND, VEC, THREADS, false>), grid, block, lds, s, a);
    return hipGetLastError();
}
template <int KIND>
static hipError_t launch_probe_kind(bool direct, StepShape shape, const StepArgs& a, int64_t n_blocks, hipStream_t s) {
    if (shape == StepShape::kSmall) return launch_probe_variant<KIND, StepShape::kSmall>(direct, a, n_blocks, s);
    if constexpr (KIND != 0) {
        if (shape == StepShape::kWide) return launch_probe_variant<KIND, StepShape::kWide>(direct, a, n_blocks, s);
    }
    return launch_probe_variant<KIND, StepShape::kUsual>(direct, a, n_blocks, s);
}
hipError_t launch_probe(int kind, bool direct, StepShape shape, const StepArgs& a, int64_t n_blocks, hipStream_t s) {
    if (kind == 0) return launch_probe_kind<0>(direct, shape, a, n_blocks, s);
    return kind == 1 ? launch_probe_kind<1>(direct, shape, a, n_blocks, s) : launch_probe_kind<2>(direct, shape, a, n_blocks, s);
}

// ------------------------------------------------------------ clock monitor --
//
// A measurement aid: ONE lane samples the shader clock while other kernels run.  Each sample spans
// ticks_per_sample ticks of the fixed-frequency counter (wall_clock64) and stores how many ticks and how many
// shader-clock cycles (clock64) went by; cycles / ticks x tick rate is the clock the compute units ran at
// in that interval.  The wait is bounded, so the kernel ends by itself after n_samples samples at the latest.
__global__ __launch_bounds__(64) void clock_monitor_kernel(unsigned long long* samples, int n_samples,
                                                           unsigned long long ticks_per_sample) {
    if (threadIdx.x != 0) return;
    for (int s = 0; s < n_samples; ++s) {
        const unsigned long long r0 = wall_clock64(), c0 = clock64();
        for (int it = 0; it < (1 << 22); ++it) {
            if (wall_clock64() - r0 >= ticks_per_sample) break;
            __builtin_amdgcn_s_sleep(8);
        }
        samples[2 * s] = wall_clock64() - r0;
        samples[2 * s + 1] = clock64() - c0;
    }
}
hipError_t launch_clock_monitor(unsigned long long* samples, int n_samples, unsigned long long ticks_per_sample,
                                hipStream_t s) {
    hipLaunchKernelGGL(clock_monitor_kernel, dim3(1), dim3(64), 0, s, samples, n_samples, ticks_per_sample);
    return hipGetLastError();
}

// -------------------------------------------------------- standalone codecs --
//
// Not on the per-step path (used at initialisation, for inspection and by tests).  Every one of them has an FP32
// array on one side, and that array is most of the traffic, so the lane layout follows it: a lane owns four
// consecutive elements per pass, one 128-bit FP32 access, 64 bits of BF16 or 32 bits of codes, and a wavefront's
// access covers whole cache lines of every stream.  A quantisation group is eight lanes.  A workgroup of 256 lanes
// covers kCodecTile consecutive elements in passes of 1024, all of whose loads are issued before the first use; split and
// reconstruct take single wavefronts (below).
// Bound: HBM.  (Eight consecutive elements per lane, so two FP32 accesses that each cover half of every line and no
// non-temporal hint: 150 M elements split 174 us and, with the kernels of that time, 163 with four; reconstruct 191 and 163,
// quantize 123 and 117, dequantize 146 and 119.)

constexpr int kCodecVec = 4;
constexpr int kCodecPass = kThreads * kCodecVec;          // elements per pass
constexpr int kCodecPasses = 2;
constexpr int kCodecTile = kCodecPass * kCodecPasses;     // elements per workgroup
constexpr int kWaveThreads = 64;                          // split and reconstruct
constexpr int kWaveTile = kWaveThreads * kCodecVec;

struct LanePos {
    int64_t tile0;       // first element of the pass, or of the wavefront's part of it (wave-uniform)
    uint32_t lane_el;    // first element of the lane, from there on
    int cnt;             // elements of the lane that exist: kCodecVec, or fewer at the ragged end
};
// FULL: every element of the pass exists (known at compile time, so that no case distinction is left).
// DEALT: tile0 is where the wavefront's part begins.
template <bool FULL, bool DEALT = false>
__device__ __forceinline__ LanePos lane_pos_at(int64_t tile0, int64_t n) {
    LanePos L;
    L.tile0 = tile0;
    L.lane_el = (uint32_t)(DEALT ? threadIdx.x & 63 : threadIdx.x) * kCodecVec;
    const int64_t left = n - tile0 - (int64_t)L.lane_el;
    L.cnt = (FULL || left >= kCodecVec) ? kCodecVec : (left > 0 ? (int)left : 0);
    return L;
}

// The elements of a lane from / to an array of 4-, 2- or 1-byte elements.  Full lanes use
// vector accesses; ragged lanes go element by element and read missing elements as zero.
__device__ __forceinline__ void load_f32(float (&f)[kCodecVec], const float* p, const LanePos& L) {
    if (L.cnt == kCodecVec) {
        gld_floats(f, gbase(p, 4 * L.tile0), 4u * block_local(L.lane_el));
    } else if (L.cnt > 0) {
        load_elements(f, p + L.tile0 + L.lane_el, L.cnt);
    } else {
#pragma unroll
        for (int i = 0; i < kCodecVec; ++i) f[i] = 0.0f;
    }
}
template <bool THROUGH>
__device__ __forceinline__ void store_f32(float* p, const LanePos& L, const float (&f)[kCodecVec]) {
    if (L.cnt == kCodecVec) {
        gst_floats<THROUGH>(gbase(p, 4 * L.tile0), 4u * block_local(L.lane_el), f);
    } else {
        const auto q = as_global(p) + L.tile0 + L.lane_el;
#pragma unroll
        for (int i = 0; i < kCodecVec; ++i) if (i < L.cnt) q[i] = f[i];
    }
}
__device__ __forceinline__ void load_u16(uint32_t (&w)[kCodecVec / 2], const void* p, const LanePos& L) {
    if (L.cnt == kCodecVec) {
        gld_words(w, gbase(p, 2 * L.tile0), 2u * block_local(L.lane_el));
    } else if (L.cnt > 0) {
        uint16_t e[kCodecVec];
        load_elements(e, reinterpret_cast<const uint16_t*>(p) + L.tile0 + L.lane_el, L.cnt);
        pack_elements(w, e);
    } else {
#pragma unroll
        for (int j = 0; j < kCodecVec / 2; ++j) w[j] = 0;
    }
}
template <bool THROUGH>
__device__ __forceinline__ void store_u16(void* p, const LanePos& L, const uint32_t (&w)[kCodecVec / 2]) {
    if (L.cnt == kCodecVec) {
        gst_words<THROUGH>(gbase(p, 2 * L.tile0), 2u * block_local(L.lane_el), w);
    } else {
        const auto q = as_global(reinterpret_cast<uint16_t*>(p)) + L.tile0 + L.lane_el;
#pragma unroll
        for (int i = 0; i < kCodecVec; ++i) if (i < L.cnt) q[i] = (uint16_t)(w[i >> 1] >> (16 * (i & 1)));
    }
}
__device__ __forceinline__ void load_u8(uint32_t (&w)[kCodecVec / 4], const void* p, const LanePos& L) {
    if (L.cnt == kCodecVec) {
        gld_words(w, gbase(p, L.tile0), block_local(L.lane_el));
    } else if (L.cnt > 0) {
        uint8_t e[kCodecVec];
        load_elements(e, reinterpret_cast<const uint8_t*>(p) + L.tile0 + L.lane_el, L.cnt);
        pack_elements(w, e);
    } else {
#pragma unroll
        for (int j = 0; j < kCodecVec / 4; ++j) w[j] = 0;
    }
}
template <bool THROUGH>
__device__ __forceinline__ void store_u8(void* p, const LanePos& L, const uint32_t (&w)[kCodecVec / 4]) {
    if (L.cnt == kCodecVec) {
        gst_words<THROUGH>(gbase(p, L.tile0), block_local(L.lane_el), w);
    } else {
        const auto q = as_global(reinterpret_cast<uint8_t*>(p)) + L.tile0 + L.lane_el;
#pragma unroll
        for (int i = 0; i < kCodecVec; ++i) if (i < L.cnt) q[i] = (uint8_t)(w[i >> 2] >> (8 * (i & 3)));
    }
}
__device__ __forceinline__ uint32_t byte_of(const uint32_t (&w)[kCodecVec / 4], int i) {
    return (w[i >> 2] >> (8 * (i & 3))) & 0xffu;
}
__device__ __forceinline__ uint32_t half_of(const uint32_t (&w)[kCodecVec / 2], int i) {
    return (w[i >> 1] >> (16 * (i & 1))) & 0xffffu;
}
// A lane's small integers -> packed bytes / packed 16-bit fields (two's complement).
__device__ __forceinline__ void pack_u8(uint32_t (&w)[kCodecVec / 4], const uint32_t (&c)[kCodecVec]) {
#pragma unroll
    for (int j = 0; j < kCodecVec / 4; ++j) w[j] = pack_low_bytes(c[4 * j], c[4 * j + 1], c[4 * j + 2], c[4 * j + 3]);
}
__device__ __forceinline__ void pack_u16(uint32_t (&w)[kCodecVec / 2], const uint32_t (&c)[kCodecVec]) {
#pragma unroll
    for (int j = 0; j < kCodecVec / 2; ++j) w[j] = (c[2 * j] & 0xffffu) | (c[2 * j + 1] << 16);
}

// C and C^-1 for a correction of N = 127 (INT8) or N = 32767 (INT16) levels per side,
// written out plainly (Algorithm 1; for N = 127 the step kernels use the short forms above where they apply).
template <int N>
__device__ __forceinline__ int split_rho(float theta, uint32_t b) {
    const int E = (int)((b >> 7) & 0xffu);
    if (E == 255) return 0;                                   // non-finite theta': no correction
    const float e = theta - u2f(b << 16);
    const float en = ldexpf(e, 135 - (E < 1 ? 1 : E));        // e * 2^-l, exact
    const float c = __builtin_amdgcn_fmed3f(en, -1.0f, 1.0f);
    return (int)rintf(c * (float)N);
}
template <int N>
__device__ __forceinline__ float reconstruct_n(uint32_t b, int rho) {
    const float base = u2f(b << 16);
    if (((b >> 7) & 0xffu) == 255u) return base;
    const float q = (float)rho / (float)N;
    return base + ldexpf(q, half_ulp_log2(b));
}
// The 8-bit case given q = rho / 127.
__device__ __forceinline__ float reconstruct_q(uint32_t b, float q) {
    const float base = u2f(b << 16);
    if (((b >> 7) & 0xffu) == 255u) return base;
    return base + ldexpf(q, half_ulp_log2(b));
}

// The "directional" reading of ULP(theta'), for the experiment of Section 4.4 only.  The BF16 grid is twice
// as fine just below a power of two as above it, so for theta' = +-2^k (mantissa field 0, exponent field
// at least 2) with theta on the side of zero the values that round to theta' span a quarter of the upper
// spacing, not a half.  This reading takes the spacing of the side on which theta lies; the decoder knows
// the side from the signs of rho and theta'.  With a 16-bit correction it reproduces the fraction of
// bit-exact reconstructions that Section 4.4 prints.
__device__ __forceinline__ bool finer_side(uint32_t b, bool toward_negative) {
    const bool pow2 = (b & 0x7fu) == 0u && ((b >> 7) & 0xffu) >= 2u;
    return pow2 && (toward_negative != ((b & 0x8000u) != 0u));
}
template <int N>
__device__ __forceinline__ int split_rho_directional(float theta, uint32_t b) {
    const int E = (int)((b >> 7) & 0xffu);
    if (E == 255) return 0;
    const float e = theta - u2f(b << 16);
    const int shift = 135 - (E < 1 ? 1 : E) + ((e != 0.0f && finer_side(b, e < 0.0f)) ? 1 : 0);
    const float c = __builtin_amdgcn_fmed3f(ldexpf(e, shift), -1.0f, 1.0f);
    return (int)rintf(c * (float)N);
}
template <int N>
__device__ __forceinline__ float reconstruct_directional(uint32_t b, int rho) {
    const float base = u2f(b << 16);
    if (((b >> 7) & 0xffu) == 255u) return base;
    const float q = (float)rho / (float)N;
    return base + ldexpf(q, half_ulp_log2(b) - ((rho != 0 && finer_side(b, rho < 0)) ? 1 : 0));
}

// The rho half of C without the tables: the same three operations as split_rho, of which the clamp is the
// identity for a finite theta' (|e| <= half an ULP under round-to-nearest), with Round() as one addition.
// For N = 127 the product with N is exact (at most 16 + 7 significant bits).  A non-finite theta' gives 0.
template <int N>
__device__ __forceinline__ uint32_t split_rho_bits(float theta, uint32_t b) {
    const int E = (int)((b >> 7) & 0xffu);
    const float e = theta - u2f(b << 16);
    const float y = ldexpf(e, 135 - (E < 1 ? 1 : E)) * (float)N;
    return E == 255 ? 0u : round_to_int_bits(y);
}

// C and C^-1 as workgroups of one wavefront with one access to each stream: nothing is staged and nothing is shared, so a
// wavefront starts, moves its 256 elements and makes room for the next.  us, 256 lanes in two passes (the decoder with rho / 127
// from a staged table) -> this: split of 12 M / 38 M / 100 M elements 14.9 / 42.0 / 109.9 -> 14.2 / 40.1 / 102.3 (6.8 TB/s),
// reconstruct 15.6 / 43.0 / 108.1 -> 14.3 / 40.2 / 103.0.  Two passes per wavefront: 14.9 / 41.6 / 106.6.  The quantisers, which
// compute more, are better off as they are (momentum, 38 M: 31.2, as single wavefronts 34.5 with one pass and 31.4 with two).
template <int N, typename RHO, bool THROUGH, bool FULL>
__device__ __forceinline__ void split_tile(const float* theta, uint16_t* param, RHO* rho, int64_t n, int64_t tile0) {
    float th[kCodecVec];
    const LanePos L = lane_pos_at<FULL>(tile0, n);
    load_f32(th, theta, L);
    uint32_t pw[kCodecVec / 2], c[kCodecVec];
#pragma unroll
    for (int j = 0; j < kCodecVec / 2; ++j) pw[j] = bf16_pack(th[2 * j], th[2 * j + 1]);
#pragma unroll
    for (int i = 0; i < kCodecVec; ++i) c[i] = split_rho_bits<N>(th[i], half_of(pw, i));
    store_u16<THROUGH>(param, L, pw);
    if constexpr (sizeof(RHO) == 1) {
        uint32_t rw[kCodecVec / 4];
        pack_u8(rw, c);
        store_u8<THROUGH>(rho, L, rw);
    } else {
        uint32_t rw[kCodecVec / 2];
        pack_u16(rw, c);
        store_u16<THROUGH>(rho, L, rw);
    }
}
template <int N, typename RHO, bool THROUGH>
__global__ __launch_bounds__(kWaveThreads) void split_kernel(const float* theta, uint16_t* param, RHO* rho, int64_t n) {
    const int64_t tile0 = (int64_t)blockIdx.x * kWaveTile;
    if (n - tile0 >= kWaveTile) split_tile<N, RHO, THROUGH, true>(theta, param, rho, n, tile0);
    else split_tile<N, RHO, THROUGH, false>(theta, param, rho, n, tile0);
}

template <int N, typename RHO, bool THROUGH, bool FULL>
__device__ __forceinline__ void reconstruct_tile(const uint16_t* param, const RHO* rho, float* theta, int64_t n,
                                                 int64_t tile0) {
    static_assert(sizeof(RHO) != 1 || N == 127, "code_over_127 is for INT8 corrections");
    uint32_t pw[kCodecVec / 2], rw[sizeof(RHO) == 1 ? kCodecVec / 4 : kCodecVec / 2];
    const LanePos L = lane_pos_at<FULL>(tile0, n);
    load_u16(pw, param, L);
    if constexpr (sizeof(RHO) == 1) load_u8(rw, rho, L);
    else load_u16(rw, rho, L);
    float th[kCodecVec];
#pragma unroll
    for (int i = 0; i < kCodecVec; ++i) {
        if constexpr (sizeof(RHO) == 1) th[i] = reconstruct_q(half_of(pw, i), code_over_127(byte_of(rw, i)));
        else th[i] = reconstruct_n<N>(half_of(pw, i), (int)(int16_t)half_of(rw, i));
    }
    store_f32<THROUGH>(theta, L, th);
}
template <int N, typename RHO, bool THROUGH>
__global__ __launch_bounds__(kWaveThreads) void reconstruct_kernel(const uint16_t* param, const RHO* rho, float* theta,
                                                                   int64_t n) {
    const int64_t tile0 = (int64_t)blockIdx.x * kWaveTile;
    if (n - tile0 >= kWaveTile) reconstruct_tile<N, RHO, THROUGH, true>(param, rho, theta, n, tile0);
    else reconstruct_tile<N, RHO, THROUGH, false>(param, rho, theta, n, tile0);
}

// The data-independent experiment of Section 4.4: FP32 bit patterns first, first + stride, ...
// (below 2^32) go through C then C^-1; errors are measured in double.  Statistics layout
// (doubles): [0] values measured, [1] skipped (non-finite theta or theta'), [2] values with
// |theta - theta'| > ULP(theta')/2, [3] max |theta_hat - theta| / (ULP(theta')/(4N)),
// [4] max relative error over normal theta, [5] bit-exact reconstructions, [6] rho outside
// [-N, N], [7] unused, [8 + E] sum of relative errors, [264 + E] count and [520 + E] bit-exact
// reconstructions of the normal values with FP32 exponent field E.  [3] and [4] are accumulated as the
// bit patterns of non-negative doubles with an integer maximum.  DIRECTIONAL selects the alternative
// reading of ULP(theta') above; [2] and [3] are measured against the printed (literal) ULP in both cases.
constexpr int kSweepPerLane = 256;

template <int N, bool DIRECTIONAL>
__global__ __launch_bounds__(kThreads) void sweep_kernel(uint64_t first, uint64_t stride, uint64_t count,
                                                         double* st) {
    __shared__ double bin_sum[256];
    __shared__ double bin_cnt[256];
    __shared__ double bin_exact[256];
    bin_sum[threadIdx.x] = 0.0;
    bin_cnt[threadIdx.x] = 0.0;
    bin_exact[threadIdx.x] = 0.0;
    __syncthreads();
    const uint64_t j0 = ((uint64_t)blockIdx.x * kThreads + threadIdx.x) * kSweepPerLane;
    double measured = 0, skipped = 0, viol = 0, exact = 0, range_bad = 0, max_ratio = 0, max_rel = 0;
    double run_sum = 0, run_cnt = 0, run_exact = 0;
    int run_exp = -1;
    for (int k = 0; k < kSweepPerLane; ++k) {
        const uint64_t j = j0 + (uint64_t)k;
        if (j >= count) break;
        const uint32_t bits = (uint32_t)(first + j * stride);
        const float theta = u2f(bits);
        const uint32_t Ef = (bits >> 23) & 0xffu;
        if (Ef == 255u) { skipped += 1; continue; }
        const uint32_t b = bf16_pack(theta, 0.0f) & 0xffffu;
        if (((b >> 7) & 0xffu) == 255u) { skipped += 1; continue; }
        const int rho = DIRECTIONAL ? split_rho_directional<N>(theta, b) : split_rho<N>(theta, b);
        const float hat = DIRECTIONAL ? reconstruct_directional<N>(b, rho) : reconstruct_n<N>(b, rho);
        measured += 1;
        const double th = (double)theta, tp = (double)u2f(b << 16);
        int E = (int)((b >> 7) & 0xffu);
        E = E < 1 ? 1 : E;
        const double u = ldexp(1.0, E - 134);
        if (fabs(th - tp) > 0.5 * u) viol += 1;
        const double err = fabs((double)hat - th);
        const double ratio = err / (u / (4.0 * N));
        max_ratio = ratio > max_ratio ? ratio : max_ratio;
        if (hat == theta) exact += 1;
        if (rho < -N || rho > N) range_bad += 1;
        if (Ef >= 1u) {
            const double rel = err / fabs(th);
            max_rel = rel > max_rel ? rel : max_rel;
            if ((int)Ef != run_exp) {
                if (run_cnt > 0) {
                    atomicAdd(&bin_sum[run_exp], run_sum); atomicAdd(&bin_cnt[run_exp], run_cnt);
                    atomicAdd(&bin_exact[run_exp], run_exact);
                }
                run_exp = (int)Ef; run_sum = 0; run_cnt = 0; run_exact = 0;
            }
            run_sum += rel; run_cnt += 1;
            if (hat == theta) run_exact += 1;
        }
    }
    if (run_cnt > 0) {
        atomicAdd(&bin_sum[run_exp], run_sum); atomicAdd(&bin_cnt[run_exp], run_cnt);
        atomicAdd(&bin_exact[run_exp], run_exact);
    }
    if (measured > 0) atomicAdd(&st[0], measured);
    if (skipped > 0) atomicAdd(&st[1], skipped);
    if (viol > 0) atomicAdd(&st[2], viol);
    if (exact > 0) atomicAdd(&st[5], exact);
    if (range_bad > 0) atomicAdd(&st[6], range_bad);
    atomicMax(reinterpret_cast<unsigned long long*>(&st[3]), (unsigned long long)__double_as_longlong(max_ratio));
    atomicMax(reinterpret_cast<unsigned long long*>(&st[4]), (unsigned long long)__double_as_longlong(max_rel));
    __syncthreads();
    if (bin_cnt[threadIdx.x] > 0) {
        atomicAdd(&st[8 + threadIdx.x], bin_sum[threadIdx.x]);
        atomicAdd(&st[264 + threadIdx.x], bin_cnt[threadIdx.x]);
        atomicAdd(&st[520 + threadIdx.x], bin_exact[threadIdx.x]);
    }
}

// Group quantizers.  LINEAR drops the compander (the plain absmax-scaled integer quantisation that Section 4.5
// takes as its baseline): momentum code = Round(127 m / s), variance code = Round(255 v / s) with s the group
// maximum of v itself.
//
// The companded codes are decided from an estimate, as in the step kernels: with their exact form (an IEEE division
// or square root per element) throughout, 150 M elements of m / v took 120 / 125 us, with the estimate 117 / 118
// (6.5 TB/s).  Momentum: below.  Variance: y* = v_sqrt_f32(v) * RN(255 r), where the hardware root is
// within one ulp (flashoptim_selftest, section 1).  In units of 2^-24 the estimate is off by 2 (root) + 1 (255 r) and
// the exact argument of Round() by 3 (root, * r, * 255): 6 * 2^-24 * 255.5 < 9.2e-5, and the fused multiply-add that
// forms y* -+ w rounds by at most 2^-17 = 7.7e-6, so w = 1.1e-4 decides.  A subnormal v has y below 1e-9 for every FP16
// scale, far from a tie.
constexpr float kTieWindowCodecV = 1.1e-4f;

// The momentum codes' estimate without the reciprocal of the scale: y = 254 f(m / s) with f(x) = x / (1 + |x|), which is
// 254 m / (s + |m|).  Errors relative to 254 f, in units of 2^-24.  The exact chain: r and m1 (1 each, times the sensitivity
// 1 / (1 + |x|) of f), den, m2 and the product with 127 (1 each).  The estimate: s + |m| (1), v_rcp_f32 (1 ulp: 2).  At
// |x| = 1, where it is largest, 7 * 2^-24 * 127 = 5.3e-5 (beyond |x| = 1.008 the clamp holds).  The two fused multiply-adds
// round by half an ulp of a value below 1, times 254, and of one below 256: 7.6e-6 each.  So 6.9e-5 decides.
// den0 is the scale, or infinity in place of 0: p is then 1/2 and the code 0.  |m| has to stay below kCodeEstimateHi, so that
// the reciprocal is a normal number; callers take the exact form otherwise.
// Eight instructions per element become seven, and a lane's four elements share five less: the quantisation error of 16 M
// elements 25.3 -> 24.9 us, of 100 M 80.9 -> 78.6.  (Not in the steps: AdamW over 2 M elements 6.57 -> 6.46 us and the
// Llama-3.1-8B list 0 to 0.6 % faster, but flat 3.4 to 4.1 M elements, where every workgroup is resident at once, up to 3 %
// slower.)
constexpr float kTieWindowCodecM = 8.0e-5f;
constexpr float kCodeEstimateHi = 1.2676506002282294e30f;      // 2^100
__device__ __forceinline__ float code_den0(float s) { return s == 0.0f ? __builtin_inff() : s; }
__device__ __forceinline__ void m_code_bracket_of_scale(float m, float den0, float* lo, float* hi) {
    const float rc = __builtin_amdgcn_rcpf(den0 + fabsf(m));
    const float p = __builtin_amdgcn_fmed3f(fmaf(m, rc, 0.5f), 0.0f, 1.0f);
    *lo = fmaf(p, 254.0f, 1.0f - kTieWindowCodecM);
    *hi = fmaf(p, 254.0f, 1.0f + kTieWindowCodecM);
}

// quantize_lane: the codes of a lane, one byte each, and the FP16 scale bits of its group.  All eight lanes of
// a group must call it together; elements past the end are zero and do not raise the maximum.
// The group maximum of sqrt(v) is the square root of the maximum of v (the root is monotone).
template <bool VARIANCE, bool LINEAR>
__device__ __forceinline__ uint32_t quantize_lane(const float (&x)[kCodecVec], uint32_t (&w)[kCodecVec / 4]) {
    static_assert(kCodecVec == 4, "one word of codes");
    float a = 0.0f;
#pragma unroll
    for (int i = 0; i < kCodecVec; ++i) a = fmaxf(a, VARIANCE ? x[i] : fabsf(x[i]));
    a = group_max<kCodecVec>(a);
    if (VARIANCE && !LINEAR) a = sqrtf(a);
    float s;
    const uint32_t sbits = group_scale(a, &s);
    uint32_t c[kCodecVec];
    if (!LINEAR) {
        uint32_t lo_w = 0, hi_w = 0;
        const float r255 = VARIANCE ? 255.0f * recip_of_scale(s) : 0.0f, den0 = code_den0(s);
        const bool beyond = !VARIANCE && a > kCodeEstimateHi;
#pragma unroll
        for (int i = 0; i < kCodecVec; ++i) {
            float lo, hi;
            if (VARIANCE) {
                const float root = __builtin_amdgcn_sqrtf(x[i]);
                lo = fmaf(root, r255, -kTieWindowCodecV);
                hi = fmaf(root, r255, kTieWindowCodecV);
            } else {
                m_code_bracket_of_scale(x[i], den0, &lo, &hi);
            }
            lo_w = put_u8(lo, i, lo_w);
            hi_w = put_u8(hi, i, hi_w);
        }
        w[0] = VARIANCE ? lo_w : lo_w ^ 0x80808080u;
        if (any_lane((lo_w != hi_w) | beyond)) {
            const float r = recip_of_scale(s);
#pragma unroll
            for (int i = 0; i < kCodecVec; ++i) c[i] = VARIANCE ? v_code_exact(x[i], r) : m_code_exact(x[i], r);
            w[0] = pack_low_bytes(c[0], c[1], c[2], c[3]);
        }
    } else {
        const float r = recip_of_scale(s);
#pragma unroll
        for (int i = 0; i < kCodecVec; ++i) {
            c[i] = VARIANCE ? round_to_int_bits(__builtin_amdgcn_fmed3f((x[i] * r) * 255.0f, 0.0f, 255.0f))
                            : round_to_int_bits(__builtin_amdgcn_fmed3f((x[i] * r) * 127.0f, -127.0f, 127.0f));
        }
        w[0] = pack_low_bytes(c[0], c[1], c[2], c[3]);
    }
    return sbits;
}

// Decoders of Algorithms 2 and 3 (and of the linear baseline).  What is multiplied by the group scale
// is a function of the code byte alone: q / 255, q / 127, phi_m^-1(q / 127).  dequantize_byte forms it (the second division has
// a denominator in [0.99, 2] and a numerator that is 0 or at least 1 / 127); where a workgroup decodes enough to stage a
// copy of the table of these divisions (the quantisation error) dequantize_one reads it there.  The dequantiser
// with the table took 6.2 us for 5 M momentum codes (5.0 without), 30.9 (31.0) for 38 M and 77.5 (77.0) for 100 M; variance
// codes, 38 M, 31.3 (30.5).
template <bool VARIANCE, bool LINEAR>
__device__ __forceinline__ float dequantize_byte(uint32_t q, float s) {
    float c;
    if (VARIANCE) {
        c = code_over_255(q);
    } else {
        const float z = code_over_127(q);
        c = LINEAR ? z : div_rn_midrange(z, 2.0f - fabsf(z));
    }
    const float f = c * s;
    return (VARIANCE && !LINEAR) ? f * f : f;
}
template <bool VARIANCE, bool LINEAR>
__device__ __forceinline__ const float* decode_table() {
    return VARIANCE ? g_decode_tables.v : (LINEAR ? g_decode_tables.rho : g_decode_tables.m);
}
template <bool VARIANCE, bool LINEAR>
__device__ __forceinline__ float dequantize_one(const float* tab, uint32_t q, float s) {
    const float f = tab[q] * s;
    return (VARIANCE && !LINEAR) ? f * f : f;
}

__device__ __forceinline__ bool group_leader(const LanePos& L) {
    return (threadIdx.x & (kGroup / kCodecVec - 1)) == 0 && L.cnt > 0;
}

template <bool VARIANCE, bool LINEAR, bool THROUGH, bool FULL>
__device__ __forceinline__ void quantize_tile(const float* x, uint8_t* q, uint16_t* scale, int64_t n, int64_t tile0) {
    float v[kCodecPasses][kCodecVec];
#pragma unroll
    for (int r = 0; r < kCodecPasses; ++r) load_f32(v[r], x, lane_pos_at<FULL>(tile0 + r * kCodecPass, n));
#pragma unroll
    for (int r = 0; r < kCodecPasses; ++r) {
        const LanePos L = lane_pos_at<FULL>(tile0 + r * kCodecPass, n);
        uint32_t w[kCodecVec / 4];
        const uint32_t sbits = quantize_lane<VARIANCE, LINEAR>(v[r], w);
        if (L.cnt > 0) store_u8<THROUGH>(q, L, w);
        if (group_leader(L)) as_global(scale)[(L.tile0 + L.lane_el) >> 5] = (uint16_t)sbits;
    }
}
template <bool VARIANCE, bool LINEAR, bool THROUGH>
__global__ __launch_bounds__(kThreads) void quantize_kernel(const float* x, uint8_t* q, uint16_t* scale,
                                                            int64_t n) {
    const int64_t tile0 = (int64_t)blockIdx.x * kCodecTile;
    if (n - tile0 >= kCodecTile) quantize_tile<VARIANCE, LINEAR, THROUGH, true>(x, q, scale, n, tile0);
    else quantize_tile<VARIANCE, LINEAR, THROUGH, false>(x, q, scale, n, tile0);
}

__device__ __forceinline__ float load_scale(const uint16_t* scale, const LanePos& L) {
    return L.cnt > 0 ? (float)__builtin_bit_cast(_Float16, (uint16_t)as_global(scale)[(L.tile0 + L.lane_el) >> 5]) : 0.0f;
}

template <bool VARIANCE, bool LINEAR, bool THROUGH, bool FULL>
__device__ __forceinline__ void dequantize_tile(const uint8_t* q, const uint16_t* scale, float* x, int64_t n,
                                                int64_t tile0) {
    uint32_t w[kCodecPasses][kCodecVec / 4];
    float s[kCodecPasses];
#pragma unroll
    for (int r = 0; r < kCodecPasses; ++r) {
        const LanePos L = lane_pos_at<FULL>(tile0 + r * kCodecPass, n);
        load_u8(w[r], q, L);
        s[r] = load_scale(scale, L);
    }
#pragma unroll
    for (int r = 0; r < kCodecPasses; ++r) {
        const LanePos L = lane_pos_at<FULL>(tile0 + r * kCodecPass, n);
        float v[kCodecVec];
#pragma unroll
        for (int i = 0; i < kCodecVec; ++i) v[i] = dequantize_byte<VARIANCE, LINEAR>(byte_of(w[r], i), s[r]);
        store_f32<THROUGH>(x, L, v);
    }
}
template <bool VARIANCE, bool LINEAR, bool THROUGH>
__global__ __launch_bounds__(kThreads) void dequantize_kernel(const uint8_t* q, const uint16_t* scale, float* x,
                                                              int64_t n) {
    const int64_t tile0 = (int64_t)blockIdx.x * kCodecTile;
    if (n - tile0 >= kCodecTile) dequantize_tile<VARIANCE, LINEAR, THROUGH, true>(q, scale, x, n, tile0);
    else dequantize_tile<VARIANCE, LINEAR, THROUGH, false>(q, scale, x, n, tile0);
}

// Quantisation error of a buffer (Section 4.5): sum (Q^-1(Q(x)) - x)^2 and sum x^2, in double.  A workgroup walks
// over tiles blockIdx.x, blockIdx.x + gridDim.x, ... and leaves its pair of partial sums in pinned memory, where the host, which
// waits for the result anyway, adds the pairs up in the order of the workgroups.  A whole call, momentum / variance, with a second kernel of
// one workgroup that added up 2048 pairs and set a flag -> now, us: 200,000 values 12.4 -> 10.1, 1 M 13.1 -> 11.3, 5 M 16.6 / 16.9 -> 15.4 / 15.5,
// 2^24 23.9 / 24.9 -> 21.3 / 22.6, 38.6 M 37.4 / 39.0 -> 34.8 / 36.7, 100 M 74.0 / 78.6 -> 71.9 / 77.5 (of which 5.6 TB/s are left, less the 10 us
// that the smallest call takes, 6.5).  What bounds the smallest is the launch and the way to the host and back; the largest, HBM.
template <int THREADS>
__device__ __forceinline__ void block_sum_pair(double& a, double& b) {
    __shared__ double part[2][THREADS / 64];
    for (int off = 32; off > 0; off >>= 1) {
        a += __shfl_down(a, off);
        b += __shfl_down(b, off);
    }
    if ((threadIdx.x & 63) == 0) {
        part[0][threadIdx.x >> 6] = a;
        part[1][threadIdx.x >> 6] = b;
    }
    __syncthreads();
    a = b = 0.0;
#pragma unroll
    for (int k = 0; k < THREADS / 64; ++k) { a += part[0][k]; b += part[1][k]; }
}
constexpr int kNmsePasses = 2;
constexpr int kNmsePass = kNmseThreads * kCodecVec, kNmseTile = kNmsePass * kNmsePasses;
// (elements past the end are zero: their code decodes to zero and they add nothing)
template <bool FULL>
__device__ __forceinline__ void nmse_load(float (&v)[kNmsePasses][kCodecVec], const float* x, int64_t n, int64_t tile0) {
#pragma unroll
    for (int r = 0; r < kNmsePasses; ++r) load_f32(v[r], x, lane_pos_at<FULL>(tile0 + r * kNmsePass, n));
}
template <bool VARIANCE, bool LINEAR>
__device__ __forceinline__ void nmse_add(const float (&v)[kNmsePasses][kCodecVec], const float* tab, double& err, double& ref) {
#pragma unroll
    for (int r = 0; r < kNmsePasses; ++r) {
        uint32_t w[kCodecVec / 4];
        const uint32_t sbits = quantize_lane<VARIANCE, LINEAR>(v[r], w);
        const float s = (float)__builtin_bit_cast(_Float16, (uint16_t)sbits);
#pragma unroll
        for (int i = 0; i < kCodecVec; ++i) {
            const double xi = (double)v[r][i];
            const double d = (double)dequantize_one<VARIANCE, LINEAR>(tab, byte_of(w, i), s) - xi;
            err = fma(d, d, err);
            ref = fma(xi, xi, ref);
        }
    }
}
template <bool VARIANCE, bool LINEAR>
__global__ __launch_bounds__(kNmseThreads) void nmse_kernel(const float* x, int64_t n, uint64_t* words, uint32_t ticket) {
    static_assert(kNmseThreads >= 256, "a lane for every entry of the table");
    __shared__ float tab[256];
    const uint32_t i = threadIdx.x & 255;
    const float entry = decode_table<VARIANCE, LINEAR>()[i];
    double err = 0.0, ref = 0.0;
    float v[kNmsePasses][kCodecVec];
    for (int64_t tile0 = (int64_t)blockIdx.x * kNmseTile; tile0 < n; tile0 += (int64_t)gridDim.x * kNmseTile) {
        if (n - tile0 >= kNmseTile) nmse_load<true>(v, x, n, tile0);
        else nmse_load<false>(v, x, n, tile0);
        if (tile0 == (int64_t)blockIdx.x * kNmseTile) {      // (the table's way to LDS, behind the first tile's loads)
            tab[i] = entry;
            __syncthreads();
        }
        nmse_add<VARIANCE, LINEAR>(v, tab, err, ref);
    }
    block_sum_pair<kNmseThreads>(err, ref);
    if (threadIdx.x < kNmseWords) {
        const uint64_t sum = (uint64_t)__double_as_longlong(threadIdx.x < 2 ? err : ref);
        const uint64_t word = nmse_word((uint32_t)(threadIdx.x & 1 ? sum >> 32 : sum), ticket);
        __hip_atomic_store(&words[(uint64_t)blockIdx.x * kNmseWords + threadIdx.x], word, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
    }
}

// launch_part(blocks, first, n) for every launch that the tiles of n elements take, `tile` of them to a workgroup of `threads` lanes:
// the n elements from `first` on.  (One launch holds fewer than 2^32 work-items.)
template <typename F>
static hipError_t for_each_launch(int64_t n, int tile, int threads, F launch_part) {
    const int64_t tiles = (n + tile - 1) / tile;
    for (int64_t t = 0, k; t < tiles; t += k) {
        k = launch_span(tiles, t, threads);
        const int64_t first = t * tile, left = n - first;
        const hipError_t e = launch_part((unsigned)k, first, left < k * tile ? left : k * tile);
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}
template <int N, typename RHO>
static hipError_t launch_split_n(const float* theta, uint16_t* param, RHO* rho, int64_t n, hipStream_t s) {
    return for_each_launch(n, kWaveTile, kWaveThreads, [=](unsigned blocks, int64_t at, int64_t count) {
        return launch(codec_through(n) ? split_kernel<N, RHO, true> : split_kernel<N, RHO, false>, blocks, kWaveThreads, 0, s, theta + at,
                      param + at, rho + at, count);
    });
}
hipError_t launch_split(int bits, const float* theta, void* param, void* rho, int64_t n, hipStream_t s) {
    return bits == 8 ? launch_split_n<127>(theta, (uint16_t*)param, (int8_t*)rho, n, s)
                     : launch_split_n<32767>(theta, (uint16_t*)param, (int16_t*)rho, n, s);
}
template <int N, typename RHO>
static hipError_t launch_reconstruct_n(const uint16_t* param, const RHO* rho, float* theta, int64_t n, hipStream_t s) {
    return for_each_launch(n, kWaveTile, kWaveThreads, [=](unsigned blocks, int64_t at, int64_t count) {
        return launch(codec_through(n) ? reconstruct_kernel<N, RHO, true> : reconstruct_kernel<N, RHO, false>, blocks, kWaveThreads, 0, s,
                      param + at, rho + at, theta + at, count);
    });
}
hipError_t launch_reconstruct(int bits, const void* param, const void* rho, float* theta, int64_t n, hipStream_t s) {
    return bits == 8 ? launch_reconstruct_n<127>((const uint16_t*)param, (const int8_t*)rho, theta, n, s)
                     : launch_reconstruct_n<32767>((const uint16_t*)param, (const int16_t*)rho, theta, n, s);
}
hipError_t launch_sweep(int bits, bool directional, uint64_t first, uint64_t stride, uint64_t count, double* stats,
                        hipStream_t s) {
    const uint64_t lanes = (count + kSweepPerLane - 1) / kSweepPerLane;
    const dim3 grid((unsigned)((lanes + kThreads - 1) / kThreads)), block(kThreads);
#define FO_SWEEP(NN, DIR) hipLaunchKernelGGL((sweep_kernel<NN, DIR>), grid, block, 0, s, first, stride, count, stats)
    if (bits == 8) { if (directional) FO_SWEEP(127, true); else FO_SWEEP(127, false); }
    else { if (directional) FO_SWEEP(32767, true); else FO_SWEEP(32767, false); }
#undef FO_SWEEP
    return hipGetLastError();
}
// Calls f(VARIANCE, LINEAR, THROUGH) with the choices as compile-time constants (std::integral_constant).
template <typename F>
static hipError_t dispatch_codec(bool variance, bool linear, bool through, F f) {
    typedef std::true_type yes;
    typedef std::false_type no;
    const auto with = [=](auto T) {
        if (variance) return linear ? f(yes(), yes(), T) : f(yes(), no(), T);
        return linear ? f(no(), yes(), T) : f(no(), no(), T);
    };
    return through ? with(yes()) : with(no());
}
hipError_t launch_quantize(bool variance, bool linear, const float* x, void* q, uint16_t* scale, int64_t n, hipStream_t s) {
    return dispatch_codec(variance, linear, codec_through(n), [=](auto V, auto L, auto T) {
        return for_each_launch(n, kCodecTile, kThreads, [=](unsigned blocks, int64_t at, int64_t count) {
            return launch(quantize_kernel<decltype(V)::value, decltype(L)::value, decltype(T)::value>, blocks, kThreads, 0, s, x + at,
                          (uint8_t*)q + at, scale + at / kGroup, count);
        });
    });
}
hipError_t launch_dequantize(bool variance, bool linear, const void* q, const uint16_t* scale, float* x, int64_t n,
                             hipStream_t s) {
    return dispatch_codec(variance, linear, codec_through(n), [=](auto V, auto L, auto T) {
        return for_each_launch(n, kCodecTile, kThreads, [=](unsigned blocks, int64_t at, int64_t count) {
            return launch(dequantize_kernel<decltype(V)::value, decltype(L)::value, decltype(T)::value>, blocks, kThreads, 0, s,
                          (const uint8_t*)q + at, scale + at / kGroup, x + at, count);
        });
    });
}
// Three workgroups to a compute unit, four for long arrays: the host reads as many pairs, which takes it some microseconds, and more
// in flight pays only where there is much to read.  With 768 / 1024 workgroups, momentum (variance), us: 5 M values 15.4 / 16.5, with 2048 21; 12 M
// 19.2 / 19.2 (20.9 / 20.8), 20 M 24.4 / 24.5 (25.9 / 25.8), 28 M 29.6 / 28.8 (31.9 / 30.6), 34 M 33.7 / 32.9 (36.3 / 35.1), 45 M 39.9 / 39.3 (43.0 /
// 41.6), 60 M 49.1 / 48.3 (54.8 / 52.4), 100 M 77.1 / 76.1 (83.7 / 81.8).  They are equal up to 20 M; from there to the line at 2^25 it costs up to 4 %.
int nmse_blocks(int64_t n) {
    const int64_t tiles = (n + kNmseTile - 1) / kNmseTile, most = n < ((int64_t)1 << 25) ? 768 : kNmseMaxBlocks;
    return (int)(tiles < most ? tiles : most);
}
hipError_t launch_nmse(bool variance, bool linear, const float* x, int64_t n, uint64_t* words, uint32_t ticket, hipStream_t s) {
    return dispatch_codec(variance, linear, false, [=](auto V, auto L, auto) {
        return launch(nmse_kernel<decltype(V)::value, decltype(L)::value>, (unsigned)nmse_blocks(n), kNmseThreads, 0, s, x, n, words, ticket);
    });
}

// ------------------------------------------------------ layout conversion --
//
// Migration between a standard FP32 optimizer state (theta, m, v: 12 B/param for AdamW) and
// the compressed layout: COMPRESS applies C, Q_m, Q_v (Algorithms 1-3) in one pass over a list;
// the other direction applies the inverses, the codes' factors formed as in the standalone decoders (with three staged tables of
// 256 factors per tile and 7 workgroups to a compute unit, now 6: 2 M elements 6.8 -> 6.5 us, 5 M 16.4 -> 15.8, 25 M 71.3 -> 70.3,
// GPT-2 342.7 -> 340.0, 300 M 843 -> 834).  Tile look-up of the step kernels, lane layout and arithmetic of the standalone codecs.
// One access of a lane to each stream: tiles of convert_chunk() elements.

template <bool HAS_V, bool THROUGH, bool FULL>
__device__ __forceinline__ void compress_tile(const TensorDev& T, int64_t tile0) {
    float th[kCodecVec], m[kCodecVec], v[kCodecVec];
    const LanePos L = lane_pos_at<FULL>(tile0, T.numel);
    load_f32(th, T.theta32, L);
    load_f32(m, T.m32, L);
    if (HAS_V) load_f32(v, T.v32, L);
    // every lane of a group takes part in the group maxima, also those past the end
    const int64_t group = (L.tile0 + L.lane_el) >> 5;
    uint32_t pw[kCodecVec / 2], c[kCodecVec], w[kCodecVec / 4];
#pragma unroll
    for (int j = 0; j < kCodecVec / 2; ++j) pw[j] = bf16_pack(th[2 * j], th[2 * j + 1]);
#pragma unroll
    for (int i = 0; i < kCodecVec; ++i) c[i] = split_rho_bits<127>(th[i], half_of(pw, i));
    pack_u8(w, c);
    if (L.cnt > 0) {
        store_u16<THROUGH>(T.param, L, pw);
        store_u8<THROUGH>(T.rho, L, w);
    }
    const uint32_t ms = quantize_lane<false, false>(m, w);
    if (L.cnt > 0) store_u8<THROUGH>(T.m_q, L, w);
    if (group_leader(L)) as_global(T.m_scale)[group] = (uint16_t)ms;
    if (HAS_V) {
        const uint32_t vs = quantize_lane<true, false>(v, w);
        if (L.cnt > 0) store_u8<THROUGH>(T.v_q, L, w);
        if (group_leader(L)) as_global(T.v_scale)[group] = (uint16_t)vs;
    }
}

template <bool HAS_V, bool THROUGH, bool FULL>
__device__ __forceinline__ void decompress_tile(const TensorDev& T, int64_t tile0) {
    uint32_t pw[kCodecVec / 2], rw[kCodecVec / 4], mw[kCodecVec / 4], vw[kCodecVec / 4];
    const LanePos L = lane_pos_at<FULL, convert_dealt(false, THROUGH)>(tile0, T.numel);
    load_u16(pw, T.param, L);
    load_u8(rw, T.rho, L);
    load_u8(mw, T.m_q, L);
    const float sm = load_scale(T.m_scale, L);
    float sv = 0.0f;
    if (HAS_V) {
        load_u8(vw, T.v_q, L);
        sv = load_scale(T.v_scale, L);
    }
    float f[kCodecVec];
#pragma unroll
    for (int i = 0; i < kCodecVec; ++i) f[i] = reconstruct_q(half_of(pw, i), code_over_127(byte_of(rw, i)));
    store_f32<THROUGH>(T.theta32, L, f);
#pragma unroll
    for (int i = 0; i < kCodecVec; ++i) f[i] = dequantize_byte<false, false>(byte_of(mw, i), sm);
    store_f32<THROUGH>(T.m32, L, f);
    if (HAS_V) {
#pragma unroll
        for (int i = 0; i < kCodecVec; ++i) f[i] = dequantize_byte<true, false>(byte_of(vw, i), sv);
        store_f32<THROUGH>(T.v32, L, f);
    }
}

template <bool HAS_V, bool COMPRESS, bool DIRECT, bool THROUGH>
__global__ __launch_bounds__(convert_threads(COMPRESS, THROUGH)) void convert_kernel(StepArgs a) {
    constexpr int kTile = convert_chunk(COMPRESS, THROUGH);
    static_assert(kTile == convert_threads(COMPRESS, THROUGH) * kCodecVec, "one access of a lane to each stream");
    TensorDev T;
    const int64_t tile = locate_tile<DIRECT>(a, T);
    const bool full = T.numel - tile * kTile >= kTile;
    const int64_t tile0 = convert_dealt(COMPRESS, THROUGH) ? wave_start<kTile / (64 * kCodecVec), 64 * kCodecVec>(tile, T.numel)
                                                           : tile * kTile;
    if constexpr (COMPRESS) {
        if (full) compress_tile<HAS_V, THROUGH, true>(T, tile0);
        else compress_tile<HAS_V, THROUGH, false>(T, tile0);
    } else {
        if (full) decompress_tile<HAS_V, THROUGH, true>(T, tile0);
        else decompress_tile<HAS_V, THROUGH, false>(T, tile0);
    }
}

hipError_t launch_convert(bool has_v, bool compress, bool direct, const StepArgs& a, int64_t n_blocks, hipStream_t s) {
    const unsigned threads = convert_threads(compress, a.through);
    const int64_t elems = n_blocks * convert_chunk(compress, a.through);
    const unsigned lds = lds_to_hold(convert_resident(compress, has_v, direct, a.through, elems), 0);
#define FO_CONV(HV, CP, DR) \
    return launch(a.through ? convert_kernel<HV, CP, DR, true> : convert_kernel<HV, CP, DR, false>, (unsigned)n_blocks, threads, lds, s, a)
    if (has_v) {
        if (compress) { if (direct) FO_CONV(true, true, true); else FO_CONV(true, true, false); }
        else { if (direct) FO_CONV(true, false, true); else FO_CONV(true, false, false); }
    } else {
        if (compress) { if (direct) FO_CONV(false, true, true); else FO_CONV(false, true, false); }
        else { if (direct) FO_CONV(false, false, true); else FO_CONV(false, false, false); }
    }
#undef FO_CONV
}

// ------------------------------------------------------------------ self-test --
//
// The step kernels replace some exactly rounded operations by shorter sequences that give
// the same bits provided the hardware estimates behave as documented (v_rcp_f32 within 1 ulp) or,
// for the square root built on v_rsq_f32, as verified here value by value.  This kernel checks
// those provisions on the device it runs on, against the plain IEEE operations:
//   section 0: recip_of_fp16(s) == 1.0f / s for every positive finite FP16 value s;
//   section 1: v_rcp_f32(d) within 1 ulp of 1.0f / d, its Newton refinement equal to 1.0f / d, and v_sqrt_f32(d) (the
//              codecs' variance codes) within 1 ulp of sqrtf(d), for every d in [1, 4): every mantissa, and for the
//              root either parity of the exponent;
//   section 2: sqrt_rn_midrange(x) == sqrtf(x) for EVERY FP32 value x of its range [2^-96, FLT_MAX];
//   section 3: momentum codes: wherever the two conversions of m_code_bracket agree, they agree with m_code_exact, for every
//              m' in [2^-13, 2) of either sign, and so do those of m_code_bracket_of_scale, with two scales (a value for
//              which any of the three decides on a wrong code fails, whether the others decide or not; otherwise
//              it counts as checked if all three decide);
//   section 4: variance codes: same for v_code_bracket against v_code_exact, over every FP32 value of
//              four binades of v, for the bias-correction pair and group scale the host passes.
//   section 5: div_rn_midrange(n, d) == n / d on 2^30 pseudo-random operand pairs with magnitudes
//              in [2^-60, 2^60] (n of either sign), plus pairs that share d across all mantissas of n.
//   section 6: div_faithful(n, d) within 1 ulp of n / d on the operand pairs of section 5.  (It fails on
//              a difference of more than one ulp; how often the faithful quotient differs from the
//              exact one at all is reported by counters[14].)
// counters[2 * section] counts checks, counters[2 * section + 1] failures.

constexpr uint64_t kSelftestSqrtCount = kSelftestSqrtValues;
constexpr uint64_t kSelftestDivCount = (1ull << 30) + (1ull << 24);
constexpr uint64_t kSelftestVarCount = 4ull * (1ull << 23);
constexpr int kSelftestPerLane = 64;

__device__ __forceinline__ uint32_t selftest_hash(uint64_t x) {
    x ^= x >> 33; x *= 0xff51afd7ed558ccdull; x ^= x >> 33; x *= 0xc4ceb9fe1a85ec53ull; x ^= x >> 33;
    return (uint32_t)x;
}

// One check of `section` on value number gid of its domain.
__device__ __forceinline__ void selftest_one(int section, uint64_t gid, const StepConsts& c, float scale_r,
                                             bool& checked, bool& failed, bool& inexact) {
    checked = false; failed = false; inexact = false;
    if (section == 0) {
        if (gid >= 1 && gid <= 0x7bffu) {
            const float s = (float)__builtin_bit_cast(_Float16, (uint16_t)gid);
            checked = true;
            failed = f2u(recip_of_fp16(s)) != f2u(1.0f / s);
        }
    } else if (section == 1) {
        if (gid < (1ull << 24)) {
            const float d = u2f(0x3f800000u + (uint32_t)gid);            // [1, 4)
            const float r0 = __builtin_amdgcn_rcpf(d);
            const int32_t diff = (int32_t)f2u(r0) - (int32_t)f2u(1.0f / d);
            const int32_t root_diff = (int32_t)f2u(__builtin_amdgcn_sqrtf(d)) - (int32_t)f2u(sqrtf(d));
            checked = true;
            failed = diff > 1 || diff < -1 || f2u(fmaf(fmaf(-d, r0, 1.0f), r0, r0)) != f2u(1.0f / d) ||
                     root_diff > 1 || root_diff < -1;
        }
    } else if (section == 2) {
        if (gid < kSelftestSqrtCount) {
            const float x = u2f(0x0f800000u + (uint32_t)gid);                     // 2^-96 ... FLT_MAX, every value
            checked = true;
            failed = f2u(sqrt_rn_midrange(x)) != f2u(sqrtf(x));
        }
    } else if (section == 3) {
        if (gid < 2ull * 14 * (1ull << 23)) {
            const uint32_t sign = (uint32_t)(gid & 1) << 31;
            const uint32_t mag = 0x39000000u + (uint32_t)(gid >> 1);     // 2^-13 ... 2
            const float m1 = u2f(sign | mag);
            float lo, hi;
            checked = true;
            const auto compare = [&](uint32_t exact) {
                const uint32_t a = put_u8(lo, 0, 0);
                if (a != put_u8(hi, 0, 0)) checked = false;
                else if ((a ^ 0x80u) != (exact & 0xffu)) failed = true;
            };
            m_code_bracket(m1, 1.0f, &lo, &hi);
            compare(m_code_exact(m1, 1.0f));
            for (int k = 0; k < 2; ++k) {
                const float s = k ? 0x1.7fcp-14f : 1.0f, m = m1 * s;
                m_code_bracket_of_scale(m, s, &lo, &hi);
                compare(m_code_exact(m, recip_of_fp16(s)));
            }
            checked |= failed;
        }
    } else if (section == 5 || section == 6) {
        if (gid < kSelftestDivCount) {
            uint32_t nb, db;
            if (gid < (1ull << 30)) {
                const uint32_t h1 = selftest_hash(2 * gid + 1), h2 = selftest_hash(2 * gid + 2);
                // exponent fields 67..187 = 2^-60 .. 2^60
                nb = (h1 & 0x807fffffu) | ((67u + (h1 >> 23) % 121u) << 23);
                db = (h2 & 0x007fffffu) | ((67u + (h2 >> 23) % 121u) << 23);
            } else {
                const uint32_t k = (uint32_t)(gid - (1ull << 30));
                nb = 0x3a000000u + (k & 0x7fffffu) + ((k >> 23) << 31);      // all mantissas, both signs
                db = 0x38d1b717u + (k >> 23) * 0x00345678u;                   // a typical denominator ~1e-4
            }
            const float n = u2f(nb), d = u2f(db);
            checked = true;
            if (section == 5) {
                failed = f2u(div_rn_midrange(n, d)) != f2u(n / d);
            } else {
                const int32_t diff = (int32_t)f2u(div_faithful(n, d)) - (int32_t)f2u(n / d);
                failed = diff > 1 || diff < -1;
                inexact = diff != 0;
            }
        }
    } else {
        if (gid < kSelftestVarCount) {
            // binades of v starting at 2^-30, 2^-29, 2^-11, 2^-10 (odd and even exponents; with the
            // scales used by the host the codes land in 6..64 and in 180..255 and beyond)
            const uint32_t k = (uint32_t)(gid >> 23), mant = (uint32_t)gid & 0x7fffffu;
            const uint32_t ebits = (k == 0 ? 97u : k == 1 ? 98u : k == 2 ? 116u : 117u) << 23;
            const float v = u2f(ebits | mant);
            const float root_hat = sqrtf(v * c.rbc2);
            const float kr255 = fmaf(c.k255_hi, scale_r, c.k255_lo * scale_r);
            float lo, hi;
            v_code_bracket(root_hat, kr255, &lo, &hi);
            const uint32_t a = put_u8(lo, 0, 0), b = put_u8(hi, 0, 0);
            const uint32_t exact = v_code_exact(v, scale_r) & 0xffu;
            checked = (a == b);
            failed = a != exact;
        }
    }
}

// A lane checks kSelftestPerLane values (number gid = first + j * lanes in the grid) and keeps its counts in
// registers; a workgroup adds them up in LDS and issues at most three global atomics.  (One atomic per
// wavefront and value made the exhaustive square-root section take 350 ms, all of it spent on the
// 29 million updates of one counter.)
__global__ __launch_bounds__(kThreads) void selftest_kernel(unsigned long long* counters, int section,
                                                            StepConsts c, float scale_r) {
    __shared__ unsigned int tally[3];
    if (threadIdx.x < 3) tally[threadIdx.x] = 0;
    __syncthreads();
    const uint64_t lanes = (uint64_t)gridDim.x * kThreads;
    uint64_t gid = (uint64_t)blockIdx.x * kThreads + threadIdx.x;
    unsigned int n_checked = 0, n_failed = 0, n_inexact = 0;
    for (int j = 0; j < kSelftestPerLane; ++j, gid += lanes) {
        bool checked, failed, inexact;
        selftest_one(section, gid, c, scale_r, checked, failed, inexact);
        n_checked += checked ? 1u : 0u;
        n_failed += (checked && failed) ? 1u : 0u;
        n_inexact += inexact ? 1u : 0u;
    }
    if (n_checked) atomicAdd(&tally[0], n_checked);
    if (n_failed) atomicAdd(&tally[1], n_failed);
    if (n_inexact) atomicAdd(&tally[2], n_inexact);
    __syncthreads();
    if (threadIdx.x == 0) {
        if (tally[0]) atomicAdd(&counters[2 * section], (unsigned long long)tally[0]);
        if (tally[1]) atomicAdd(&counters[2 * section + 1], (unsigned long long)tally[1]);
        if (tally[2]) atomicAdd(&counters[14], (unsigned long long)tally[2]);
    }
}

hipError_t launch_selftest(unsigned long long* counters, int section, const StepConsts& c, float scale_r,
                           hipStream_t s) {
    uint64_t n = 0;
    if (section == 0) n = 0x7c00;
    else if (section == 1) n = 1ull << 24;
    else if (section == 2) n = kSelftestSqrtCount;
    else if (section == 3) n = 2ull * 14 * (1ull << 23);
    else if (section == 5 || section == 6) n = kSelftestDivCount;
    else n = kSelftestVarCount;
    const uint64_t per_block = (uint64_t)kThreads * kSelftestPerLane;
    hipLaunchKernelGGL(selftest_kernel, dim3((unsigned)((n + per_block - 1) / per_block)), dim3(kThreads), 0, s,
                       counters, section, c, scale_r);
    return hipGetLastError();
}

// ----------------------------------------------------------- checkpoint copy --
//
// Gather / scatter of byte segments: each workgroup copies one piece of one segment, 16 bytes per lane (segment starts
// are 16-byte aligned on both sides), the ragged end byte by byte, and - when packing - zero-fills the padding up to
// pad_bytes.  Bound: HBM.
//
// One access per lane and 1024 lanes: pieces of 16 KB that are read and written at once and make room for the next, the
// pieces of large segments dealt out among the wavefronts of a group of workgroups (wave_part; a part is 1 KB).  In us, a pack and an unpack of
// ResNet-50 / GPT-2 / a Llama layer (SGD) / two layers with embedding: 89.2 / 407 / 555 / 3209 with every piece in one piece, 89.0 / 383 / 522 /
// 2917 (6.75 TB/s) dealt out; as pieces of 8 KB and 512 lanes 88.4 / 382 / 525 / 2925, of 4 KB 88.9 / 382 / 524 / 2938.  More accesses per lane are
// slower (in one piece, pack of GPT-2 512 lanes x 16 accesses 225, 1024 x 8 217, 1024 x 1 201).  Pieces are found as the step kernels find their
// tiles, through a coarse table and the segments themselves: a table with an entry per piece would be 20 MB for the 41 GB of Llama-3.1-8B.
//
// header: the blob's header and table when packing; the workgroup behind the last piece writes them to header_dst.
// verdict: when unpacking, what check_header_kernel has found; nothing is written unless it admits this copy.
constexpr int kCopyThreads = kCopyPiece / 16;
static_assert(kHeaderStepAt % 16 == 0, "the step is the low half of one 16-byte access");
// Whether 16 bytes of a blob's header or table, number i, are not what the list expects.  The step is the caller's.
__device__ __forceinline__ bool header_differs(uint4 x, uint4 y, uint32_t i) {
    const uint32_t d = (x.z ^ y.z) | (x.w ^ y.w);
    return (i == kHeaderStepAt / 16 ? d : d | (x.x ^ y.x) | (x.y ^ y.y)) != 0;
}
// What unpacking found, for the host that watches the flag.
__device__ __forceinline__ void report_header(const uint4* blob, bool ok, int64_t* out, uint32_t* flag, uint64_t ticket) {
    const uint4 step = blob[kHeaderStepAt / 16];
    out[0] = ok;
    out[1] = (int64_t)((uint64_t)step.y << 32 | step.x);
    __hip_atomic_store(flag, (uint32_t)ticket, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_SYSTEM);     // behind this lane's two stores
}
// The segment that holds piece b: the last one that begins there or before, among those of its coarse entry.
__device__ __forceinline__ CopySegment locate_piece(const CopyArgs& a, uint32_t b) {
    const uint32_t* entry = a.coarse + (b >> a.coarse_shift);
    uint32_t t = entry[0];
    if (a.coarse_shift) t = entry_of(b, t, entry[1], [&](uint32_t i) { return a.segs[i].first_piece; });
    return a.segs[t];
}
// The lane's offset in the segment of piece b.
__device__ __forceinline__ int64_t copy_offset(const CopySegment& sg, uint32_t b) {
    const int64_t piece = b - sg.first_piece;
    if (sg.n_pieces < kTileGroup) return piece * kCopyPiece + (int64_t)threadIdx.x * 16;      // (nothing to deal out, sooner found)
    return wave_start<kCopyThreads / 64, 64 * 16>(piece, sg.bytes) + (int64_t)(threadIdx.x & 63) * 16;
}
__device__ __forceinline__ void copy_end(const CopySegment& sg, int64_t o) {
    for (int k = 0; k < 16 && o + k < sg.pad_bytes; ++k) sg.dst[o + k] = (o + k < sg.bytes) ? sg.src[o + k] : (uint8_t)0;
}
__global__ __launch_bounds__(kCopyThreads) void copy_kernel(CopyArgs a) {
    const uint32_t b = blockIdx.x + a.piece_offset;
    const bool go = !a.verdict || verdict_admits(*a.verdict, a.ticket);      // (looked up beside the piece)
    if (b == a.n_pieces) {
        for (uint32_t i = threadIdx.x; i < a.header_n16; i += kCopyThreads) {
            uint4 v = a.header[i];
            if (i == kHeaderStepAt / 16) {
                v.x = (uint32_t)a.step;
                v.y = (uint32_t)(a.step >> 32);
            }
            a.header_dst[i] = v;
        }
        return;
    }
    const CopySegment sg = locate_piece(a, b);
    if (!go) return;
    const int64_t o = copy_offset(sg, b);
    if (o + 16 <= sg.bytes) {
        const uint4 v = ld128(sg.src + o);
        st128(sg.dst + o, v.x, v.y, v.z, v.w);
    } else {
        copy_end(sg, o);
    }
}
// The same when every workgroup checks the header for itself: its two loads stand beside that of the piece, and nothing is stored
// before all lanes have compared.  The workgroup that reports, for which the host waits, does so before it looks for its piece.
__global__ __launch_bounds__(kCopyThreads) void copy_kernel(CheckedCopyArgs a) {
    const uint32_t b = blockIdx.x + a.piece_offset, i = threadIdx.x;
    bool differs = false;
    if (i < a.header_n16) differs = header_differs(a.header[i], a.found[i], i);
    CopySegment sg;
    int64_t o = 0;
    uint4 v = make_uint4(0, 0, 0, 0);
    const auto load = [&] {
        sg = locate_piece(a, b);
        o = copy_offset(sg, b);
        if (o + 16 <= sg.bytes) v = ld128(sg.src + o);
    };
    if (b != 0) load();
    const bool ok = __syncthreads_or(differs) == 0;
    if (b == 0) {
        if (i == 0) report_header(a.found, ok, a.out, a.flag, a.ticket);
        load();
    }
    if (!ok) return;
    if (o + 16 <= sg.bytes) st128(sg.dst + o, v.x, v.y, v.z, v.w);
    else copy_end(sg, o);
}

// Consecutive launches of as many pieces as one may have: 2^22 - 1, or 64 GiB.
template <typename ARGS>
static hipError_t launch_pieces(ARGS a, int64_t total, hipStream_t s) {
    void (*kernel)(ARGS) = copy_kernel;
    for (int64_t first = 0, n; first < total; first += n) {
        n = launch_span(total, first, kCopyThreads);
        a.piece_offset = (uint32_t)first;
        const hipError_t e = launch(kernel, (unsigned)n, kCopyThreads, 0, s, a);
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}
hipError_t launch_copy(CopyArgs a, hipStream_t s) { return launch_pieces(a, (int64_t)a.n_pieces + (a.header ? 1 : 0), s); }
hipError_t launch_checked_copy(CheckedCopyArgs a, hipStream_t s) {
    if (a.n_pieces == 0 || a.header_n16 > (uint32_t)kCopyThreads) return hipErrorInvalidValue;     // (nobody would report, or compare)
    return launch_pieces(a, a.n_pieces, s);
}

// Small transfers between pinned host memory and device memory by a kernel instead of a copy command (16-byte
// multiples; bound by the link to the host), which costs the host several times a launch.
__global__ __launch_bounds__(256) void move_kernel(const uint4* src, uint4* dst, uint32_t n16) {
    for (uint32_t i = blockIdx.x * 256u + threadIdx.x; i < n16; i += gridDim.x * 256u) dst[i] = src[i];
}
hipError_t launch_move(const void* src, void* dst, size_t bytes, hipStream_t s) {
    const uint32_t n16 = (uint32_t)((bytes + 15) / 16), blocks = (n16 + 255) / 256;
    return launch(move_kernel, blocks < 64 ? blocks : 64, 256, 0, s, (const uint4*)src, (uint4*)dst, n16);
}

// Table entries from kernel arguments.  Against a pinned buffer that a kernel reads and reports as read, which the host
// then has to wait for: ResNet-50 list with other rates in every step 58.3 -> 54.9 us a step, 9 us of them on the host.
__global__ __launch_bounds__(256) void table_update_kernel(TableUpdate u, TensorDev* table) {
    const uint32_t per = update_words(u.fields);
    for (uint32_t i = threadIdx.x; i < u.count; i += 256) {
        TensorDev& t = table[u.first + i];
        uint32_t at = i * per;
        if (u.fields & kUpdateGrad) {
            t.grad = reinterpret_cast<const void*>(u.words[at] | (uint64_t)u.words[at + 1] << 32);
            at += 2;
        }
        if (u.fields & kUpdateLr) t.lr = u2f(u.words[at++]);
        if (u.fields & kUpdateWd) t.wd = u2f(u.words[at]);
    }
}
hipError_t launch_table_update(const TableUpdate& u, TensorDev* table, hipStream_t s) {
    return launch(table_update_kernel, 1, 256, 0, s, u, table);
}

// Whether a blob's header and table are what this list would have written, but for the step: *verdict tells the copy that
// follows on the stream, out[0] and the flag behind it the host, which gets the step in out[1].  (When the host compared them
// itself, the copy was launched only once it had: a pack and an unpack of ResNet-50, 131 MB each: 101.1 us, so 91.3.)
constexpr int kCheckThreads = 1024;
__global__ __launch_bounds__(kCheckThreads) void check_header_kernel(const uint4* expected, const uint4* blob, uint32_t n16,
                                                                     uint64_t* verdict, int64_t* out, uint32_t* flag,
                                                                     uint64_t ticket) {
    __shared__ uint32_t differs;
    if (threadIdx.x == 0) differs = 0;
    __syncthreads();
    bool d = false;
    for (uint32_t i = threadIdx.x; i < n16; i += kCheckThreads) d |= header_differs(expected[i], blob[i], i);
    if (d) atomicOr(&differs, 1u);
    __syncthreads();
    if (threadIdx.x != 0) return;
    *verdict = verdict_word(ticket, differs == 0);
    report_header(blob, differs == 0, out, flag, ticket);
}
hipError_t launch_check_header(const void* expected, const void* blob, size_t bytes, uint64_t* verdict, int64_t* out,
                               uint32_t* flag, uint64_t ticket, hipStream_t s) {
    return launch(check_header_kernel, 1, kCheckThreads, 0, s, (const uint4*)expected, (const uint4*)blob, (uint32_t)(bytes / 16), verdict,
                  out, flag, ticket);
}

}  // namespace fo
