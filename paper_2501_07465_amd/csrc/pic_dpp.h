// pic_dpp.h -- wavefront scans on DPP (GFX9 data-parallel primitives) for gfx950.
#pragma once
#include <hip/hip_runtime.h>

namespace pic {

// ---------------------------------------------------------------------------------------------
// Wavefront segmented inclusive scan on DPP (GFX9 data-parallel primitives): four row shifts
// within rows of 16 lanes, then the row-15 and row-31 broadcasts.  Lanes hold consecutive
// (cell-sorted) particles; a segment starts where the start node differs from the previous lane.
// The per-step "add" predicates depend only on the segment heads, so they are computed once and
// reused for every value.
// ---------------------------------------------------------------------------------------------
// Lanes whose source lies outside the row (or the wavefront) read 0, as do the rows that ROWMASK leaves
// out.  With every row enabled that is the instruction's own bound control: no register has to hold
// the 0, and the move folds into the instruction that uses it.
template <int CTRL, int ROWMASK>
__device__ __forceinline__ int dpp_i(int v)
{
    return __builtin_amdgcn_update_dpp(0, v, CTRL, ROWMASK, 0xf, ROWMASK == 0xf);
}

template <int CTRL, int ROWMASK>
__device__ __forceinline__ int dpp_r(int v)
{
    return dpp_i<CTRL, ROWMASK>(v);
}

template <int CTRL, int ROWMASK>
__device__ __forceinline__ float dpp_r(float v)
{
    return __builtin_bit_cast(float, dpp_i<CTRL, ROWMASK>(__builtin_bit_cast(int, v)));
}

template <int CTRL, int ROWMASK>
__device__ __forceinline__ double dpp_r(double v)
{
    const long long b = __builtin_bit_cast(long long, v);
    const int lo = dpp_i<CTRL, ROWMASK>((int)(b & 0xffffffffll));
    const int hi = dpp_i<CTRL, ROWMASK>((int)(b >> 32));
    return __builtin_bit_cast(double, ((long long)hi << 32) | (unsigned int)lo);
}

constexpr int kRowShl1 = 0x101;
constexpr int kRowShr1 = 0x111, kRowShr2 = 0x112, kRowShr4 = 0x114, kRowShr8 = 0x118;
constexpr int kRowBcast15 = 0x142, kRowBcast31 = 0x143;

__device__ __forceinline__ unsigned seg_masks(bool head)
{
    int f = head ? 1 : 0;
    unsigned m = 0;
    int fu;
    fu = dpp_i<kRowShr1, 0xf>(f);    if (!f) m |= 1u;  f |= fu;
    fu = dpp_i<kRowShr2, 0xf>(f);    if (!f) m |= 2u;  f |= fu;
    fu = dpp_i<kRowShr4, 0xf>(f);    if (!f) m |= 4u;  f |= fu;
    fu = dpp_i<kRowShr8, 0xf>(f);    if (!f) m |= 8u;  f |= fu;
    fu = dpp_i<kRowBcast15, 0xa>(f); if (!f) m |= 16u; f |= fu;
    fu = dpp_i<kRowBcast31, 0xc>(f); if (!f) m |= 32u;
    return m;
}

template <typename R>
__device__ __forceinline__ R seg_scan(R v, unsigned m)
{
    R t;
    t = dpp_r<kRowShr1, 0xf>(v);    if (m & 1u) v += t;
    t = dpp_r<kRowShr2, 0xf>(v);    if (m & 2u) v += t;
    t = dpp_r<kRowShr4, 0xf>(v);    if (m & 4u) v += t;
    t = dpp_r<kRowShr8, 0xf>(v);    if (m & 8u) v += t;
    t = dpp_r<kRowBcast15, 0xa>(v); if (m & 16u) v += t;
    t = dpp_r<kRowBcast31, 0xc>(v); if (m & 32u) v += t;
    return v;
}

// Segments of the in-cell deposit: runs of equal keys within groups of 2^STEPS lanes (STEPS <= 4: a group
// lies in one DPP row).  f[k] is 1 on lanes whose segment reaches 2^k lanes back (no segment starts
// on the 2^k lanes up to and with this one) and 0 elsewhere, as the factor of step k of the scan; tail
// marks the last lane of each segment.  Each factor is the one before times its own row-shifted
// copy; lanes that a shift takes from outside the row read 0, which ends their segments there.
template <int STEPS>
__device__ __forceinline__ void seg_factors(int key, float (&f)[STEPS], bool& tail)
{
    static_assert(STEPS >= 1 && STEPS <= 4, "row shifts only");
    constexpr int G = 1 << STEPS;
    const int lane = (int)(threadIdx.x & 63);
    const bool first = lane % G == 0, last = lane % G == G - 1;
    const int prev = dpp_i<kRowShr1, 0xf>(key), next = dpp_i<kRowShl1, 0xf>(key);
    tail = last || next != key;
    f[0] = first || prev != key ? 0.0f : 1.0f;
    if constexpr (STEPS > 1) f[1] = f[0] * dpp_r<kRowShr1, 0xf>(f[0]);
    if constexpr (STEPS > 2) f[2] = f[1] * dpp_r<kRowShr2, 0xf>(f[1]);
    if constexpr (STEPS > 3) f[3] = f[2] * dpp_r<kRowShr4, 0xf>(f[2]);
}

// Segmented inclusive scan of N values at once over the segments of seg_factors: step k adds the value
// 2^k lanes before times the factor f[k], for every value before step k + 1, so the DPP reads of one
// value follow the writes of the others and need no wait states.  One fused multiply-add per value and
// step: v + 1 * t rounds as v + t, v + 0 * t is v for finite values (callers add others by themselves).
template <int STEPS, int N>
__device__ __forceinline__ void seg_scan_n(double (&v)[N], const float (&f)[STEPS])
{
    double t[N];
#define PIC_SCAN_STEP(K, CTRL)                                                               \
    if constexpr (STEPS > K) {                                                               \
        const double fk = (double)f[K];                                                      \
        _Pragma("unroll") for (int q = 0; q < N; ++q) t[q] = dpp_r<CTRL, 0xf>(v[q]);         \
        _Pragma("unroll") for (int q = 0; q < N; ++q) v[q] = __builtin_fma(fk, t[q], v[q]);  \
    }
    PIC_SCAN_STEP(0, kRowShr1)
    PIC_SCAN_STEP(1, kRowShr2)
    PIC_SCAN_STEP(2, kRowShr4)
    PIC_SCAN_STEP(3, kRowShr8)
#undef PIC_SCAN_STEP
}

// FP32 form of seg_scan_n, for the N = 5, 8 and 12 deposit values of 1D, 2D and 3D: each step is one
// v_fmac_f32 per value that takes its first operand through DPP.  Written as assembly because the
// compiler does not fold a DPP move into an FMA.  Source lanes outside the row are disabled by the
// row shift (no bound_ctrl), so those lanes keep v.  A VALU write followed by a DPP read of the same
// register needs two wait states on this architecture and the compiler cannot see into the asm, so
// each step is one asm statement that starts with s_nop 1 (nothing can be scheduled between the
// wait and the reads), and the last step ends with one.
#define PIC_FM(i, f, sh) "v_fmac_f32_dpp %" #i ", %" #i ", %" #f " row_shr:" #sh " row_mask:0xf bank_mask:0xf\n\t"
#define PIC_FM5(f, sh) PIC_FM(0, f, sh) PIC_FM(1, f, sh) PIC_FM(2, f, sh) PIC_FM(3, f, sh) PIC_FM(4, f, sh)
#define PIC_FM8(f, sh) PIC_FM5(f, sh) PIC_FM(5, f, sh) PIC_FM(6, f, sh) PIC_FM(7, f, sh)
#define PIC_FM12(f, sh) PIC_FM8(f, sh) PIC_FM(8, f, sh) PIC_FM(9, f, sh) PIC_FM(10, f, sh) PIC_FM(11, f, sh)
#define PIC_V5 "+v"(v[0]), "+v"(v[1]), "+v"(v[2]), "+v"(v[3]), "+v"(v[4])
#define PIC_V8 PIC_V5, "+v"(v[5]), "+v"(v[6]), "+v"(v[7])
#define PIC_V12 PIC_V8, "+v"(v[8]), "+v"(v[9]), "+v"(v[10]), "+v"(v[11])

template <int N, int SH, bool LAST>
__device__ __forceinline__ void fmac_step(float (&v)[N], float f)
{
    static_assert(N == 5 || N == 8 || N == 12, "deposit value counts of 1D, 2D, 3D");
#define PIC_STEP_ASM(NN, sh)                                                                        \
    if constexpr (N == NN && SH == sh) {                                                            \
        if constexpr (LAST)                                                                         \
            asm volatile("s_nop 1\n\t" PIC_FM##NN(NN, sh) "s_nop 1" : PIC_V##NN : "v"(f));          \
        else                                                                                        \
            asm volatile("s_nop 1\n\t" PIC_FM##NN(NN, sh) : PIC_V##NN : "v"(f));                    \
    }
    PIC_STEP_ASM(5, 1) PIC_STEP_ASM(5, 2) PIC_STEP_ASM(5, 4) PIC_STEP_ASM(5, 8)
    PIC_STEP_ASM(8, 1) PIC_STEP_ASM(8, 2) PIC_STEP_ASM(8, 4) PIC_STEP_ASM(8, 8)
    PIC_STEP_ASM(12, 1) PIC_STEP_ASM(12, 2) PIC_STEP_ASM(12, 4) PIC_STEP_ASM(12, 8)
#undef PIC_STEP_ASM
}
#undef PIC_FM
#undef PIC_FM5
#undef PIC_FM8
#undef PIC_FM12
#undef PIC_V5
#undef PIC_V8
#undef PIC_V12

template <int STEPS, int N>
__device__ __forceinline__ void seg_scan_n(float (&v)[N], const float (&f)[STEPS])
{
    fmac_step<N, 1, STEPS == 1>(v, f[0]);
    if constexpr (STEPS > 1) fmac_step<N, 2, STEPS == 2>(v, f[1]);
    if constexpr (STEPS > 2) fmac_step<N, 4, STEPS == 3>(v, f[2]);
    if constexpr (STEPS > 3) fmac_step<N, 8, true>(v, f[3]);
}

// Plain inclusive scan over the whole wavefront (one segment starting at lane 0).
__device__ __forceinline__ unsigned scan_masks(int lane) { return seg_masks(lane == 0); }

}  // namespace pic
