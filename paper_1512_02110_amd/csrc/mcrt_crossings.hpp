// The crossings of the voxel walks, axis by axis under the lanes' own masks.
#pragma once

#include <hip/hip_runtime.h>

namespace mcrt {

// The crossings of a wavefront's walks at tn = min(tx, ty, tz): the lanes whose
// first minimum is x (then y, then z) advance their index k, their crossing
// count r and that axis' next crossing t = r g, each axis under its own lane
// mask (a compare that sets the execution mask; the lanes left go on to the
// next axis).  15
// instructions, of which the adds and multiplies take half the issue time of
// a select: per increment a select against zero and an add, and all three t
// made anew, took 16 in FP32 and 19 in FP64.  Written out because the
// compiler turns branches this short back into selects.
//
// Operands that a block writes are early-clobber ("+&v"): the y and z parts read
// inputs after the x part has written, and a caller may pass one value as both.
#define MCRT_AXIS_MASKS(EQ, X, Y, Z)                                  \
    "s_mov_b64 %[ex], exec\n\t" EQ " vcc, %[tn], %[tx]\n\t" X          \
    "s_andn2_wrexec_b64 %[no], %[ex]\n\t" EQ " vcc, %[tn], %[ty]\n\t" Y \
    "s_andn2_wrexec_b64 %[no], %[no]\n\t" Z "s_mov_b64 exec, %[ex]"
#define MCRT_CROSS(ADD, MUL, A) \
    ADD " %[r" A "], %[s" A "], %[r" A "]\n\tv_add_u32 %[k], %[k" A "], %[k]\n\t" MUL " %[t" A "], %[r" A "], %[g" A "]\n\t"
#define MCRT_CROSS_OUT                                                                                                \
    [ex] "=&s"(ex), [no] "=&s"(no), [k] "+&v"(k), [rx] "+&v"(rx), [ry] "+&v"(ry), [rz] "+&v"(rz), [tx] "+&v"(tx), \
        [ty] "+&v"(ty), [tz] "+&v"(tz)
#define MCRT_CROSS_IN                                                                                             \
    [tn] "v"(tn), [kx] "v"(kx), [ky] "v"(ky), [kz] "v"(kz), [sx] "v"(sx), [sy] "v"(sy), [sz] "v"(sz), [gx] "v"(gx), \
        [gy] "v"(gy), [gz] "v"(gz)

// LAYER: also moves the layer iz by izs on a z crossing.
template <bool LAYER, typename Real>
__device__ __forceinline__ void cross_axes(Real tn, int& k, Real& rx, Real& ry, Real& rz, Real& tx, Real& ty, Real& tz,
                                           int kx, int ky, int kz, Real sx, Real sy, Real sz, Real gx, Real gy, Real gz,
                                           int& iz, int izs) {
    unsigned long long ex, no;
    if constexpr (sizeof(Real) == 4 && !LAYER)
        asm(MCRT_AXIS_MASKS("v_cmpx_eq_f32", MCRT_CROSS("v_add_f32", "v_mul_f32", "x"),
                            MCRT_CROSS("v_add_f32", "v_mul_f32", "y"), MCRT_CROSS("v_add_f32", "v_mul_f32", "z"))
            : MCRT_CROSS_OUT
            : MCRT_CROSS_IN
            : "vcc", "scc");
    else if constexpr (sizeof(Real) == 4)
        asm(MCRT_AXIS_MASKS("v_cmpx_eq_f32", MCRT_CROSS("v_add_f32", "v_mul_f32", "x"),
                            MCRT_CROSS("v_add_f32", "v_mul_f32", "y"),
                            MCRT_CROSS("v_add_f32", "v_mul_f32", "z") "v_add_u32 %[iz], %[izs], %[iz]\n\t")
            : MCRT_CROSS_OUT, [iz] "+&v"(iz)
            : MCRT_CROSS_IN, [izs] "v"(izs)
            : "vcc", "scc");
    else if constexpr (!LAYER)
        asm(MCRT_AXIS_MASKS("v_cmpx_eq_f64", MCRT_CROSS("v_add_f64", "v_mul_f64", "x"),
                            MCRT_CROSS("v_add_f64", "v_mul_f64", "y"), MCRT_CROSS("v_add_f64", "v_mul_f64", "z"))
            : MCRT_CROSS_OUT
            : MCRT_CROSS_IN
            : "vcc", "scc");
    else
        asm(MCRT_AXIS_MASKS("v_cmpx_eq_f64", MCRT_CROSS("v_add_f64", "v_mul_f64", "x"),
                            MCRT_CROSS("v_add_f64", "v_mul_f64", "y"),
                            MCRT_CROSS("v_add_f64", "v_mul_f64", "z") "v_add_u32 %[iz], %[izs], %[iz]\n\t")
            : MCRT_CROSS_OUT, [iz] "+&v"(iz)
            : MCRT_CROSS_IN, [izs] "v"(izs)
            : "vcc", "scc");
}

// The same for a deposit's walk, whose crossings advance by an increment d.
#define MCRT_DEP(ADD, A) ADD " %[t" A "], %[d" A "], %[t" A "]\n\tv_add_u32 %[k], %[k" A "], %[k]\n\t"
template <typename Real>
__device__ __forceinline__ void dep_cross(Real tn, int& k, Real& tx, Real& ty, Real& tz, int kx, int ky, int kz,
                                          Real dtx, Real dty, Real dtz) {
    unsigned long long ex, no;
    if constexpr (sizeof(Real) == 4)
        asm(MCRT_AXIS_MASKS("v_cmpx_eq_f32", MCRT_DEP("v_add_f32", "x"), MCRT_DEP("v_add_f32", "y"),
                            MCRT_DEP("v_add_f32", "z"))
            : [ex] "=&s"(ex), [no] "=&s"(no), [k] "+&v"(k), [tx] "+&v"(tx), [ty] "+&v"(ty), [tz] "+&v"(tz)
            : [tn] "v"(tn), [kx] "v"(kx), [ky] "v"(ky), [kz] "v"(kz), [dx] "v"(dtx), [dy] "v"(dty), [dz] "v"(dtz)
            : "vcc", "scc");
    else
        asm(MCRT_AXIS_MASKS("v_cmpx_eq_f64", MCRT_DEP("v_add_f64", "x"), MCRT_DEP("v_add_f64", "y"),
                            MCRT_DEP("v_add_f64", "z"))
            : [ex] "=&s"(ex), [no] "=&s"(no), [k] "+&v"(k), [tx] "+&v"(tx), [ty] "+&v"(ty), [tz] "+&v"(tz)
            : [tn] "v"(tn), [kx] "v"(kx), [ky] "v"(ky), [kz] "v"(kz), [dx] "v"(dtx), [dy] "v"(dty), [dz] "v"(dtz)
            : "vcc", "scc");
}
// The crossings of a flight's step in two parts: first the index k and the
// crossings left c on each axis (what the next voxel's fetch needs), with the
// lanes of each axis in mx, my and mz; then, on the lanes go (of these), r and
// t of the crossed axis, the optical depth and the parameter.  Only lanes in
// on, and of them the active ones, take part.
#define MCRT_LEAVE(A) "v_add_u32 %[k], %[k" A "], %[k]\n\tv_add_u32 %[c" A "], -1, %[c" A "]\n\t"
#define MCRT_FLIGHT_LEAVE(EQ)                                                                                      \
    asm("s_mov_b64 %[ex], exec\n\ts_and_b64 exec, exec, %[on]\n\ts_mov_b64 %[mz], exec\n\t" EQ                       \
        " vcc, %[tn], %[tx]\n\ts_mov_b64 %[mx], exec\n\t" MCRT_LEAVE("x")                                           \
        "s_andn2_wrexec_b64 %[mz], %[mz]\n\t" EQ " vcc, %[tn], %[ty]\n\ts_mov_b64 %[my], exec\n\t" MCRT_LEAVE("y")  \
        "s_andn2_wrexec_b64 %[mz], %[mz]\n\t" MCRT_LEAVE("z") "s_mov_b64 exec, %[ex]"                               \
        : [ex] "=&s"(ex), [mx] "=&s"(mx), [my] "=&s"(my), [mz] "=&s"(mz), [k] "+&v"(k), [cx] "+&v"(cx), [cy] "+&v"(cy), \
          [cz] "+&v"(cz)                                                                                            \
        : [on] "s"(on), [tn] "v"(tn), [tx] "v"(tx), [ty] "v"(ty), [kx] "v"(kx), [ky] "v"(ky), [kz] "v"(kz)          \
        : "vcc", "scc")
template <typename Real>
__device__ __forceinline__ void flight_leave(unsigned long long on, Real tn, Real tx, Real ty, uint32_t& k, int& cx,
                                             int& cy, int& cz, int kx, int ky, int kz, unsigned long long& mx,
                                             unsigned long long& my, unsigned long long& mz) {
    unsigned long long ex;
    if constexpr (sizeof(Real) == 4) MCRT_FLIGHT_LEAVE("v_cmpx_eq_f32");
    else MCRT_FLIGHT_LEAVE("v_cmpx_eq_f64");
}
#undef MCRT_FLIGHT_LEAVE
#undef MCRT_LEAVE

#define MCRT_ENTER(ADD, MUL, A) \
    "s_and_b64 exec, %[m" A "], %[go]\n\t" ADD " %[r" A "], %[s" A "], %[r" A "]\n\t" MUL " %[t" A "], %[r" A "], %[g" A "]\n\t"
#define MCRT_FLIGHT_ENTER(ADD, MUL, MOV)                                                                           \
    asm("s_mov_b64 %[ex], exec\n\t" MCRT_ENTER(ADD, MUL, "x") MCRT_ENTER(ADD, MUL, "y") MCRT_ENTER(ADD, MUL, "z")  \
        "s_mov_b64 exec, %[go]\n\t" MOV " %[tau], %[taun]\n\t" MOV " %[t], %[tn]\n\ts_mov_b64 exec, %[ex]"          \
        : [ex] "=&s"(ex), [rx] "+&v"(rx), [ry] "+&v"(ry), [rz] "+&v"(rz), [tx] "+&v"(tx), [ty] "+&v"(ty), [tz] "+&v"(tz), \
          [tau] "+&v"(tau), [t] "+&v"(t)                                                                             \
        : [mx] "s"(mx), [my] "s"(my), [mz] "s"(mz), [go] "s"(go), [sx] "v"(sx), [sy] "v"(sy), [sz] "v"(sz),        \
          [gx] "v"(gx), [gy] "v"(gy), [gz] "v"(gz), [taun] "v"(taun), [tn] "v"(tn)                                 \
        : "scc")
template <typename Real>
__device__ __forceinline__ void flight_enter(unsigned long long mx, unsigned long long my, unsigned long long mz,
                                             unsigned long long go, Real& rx, Real& ry, Real& rz, Real& tx, Real& ty,
                                             Real& tz, Real sx, Real sy, Real sz, Real gx, Real gy, Real gz, Real& tau,
                                             Real taun, Real& t, Real tn) {
    unsigned long long ex;
    if constexpr (sizeof(Real) == 4) MCRT_FLIGHT_ENTER("v_add_f32", "v_mul_f32", "v_mov_b32");
    else MCRT_FLIGHT_ENTER("v_add_f64", "v_mul_f64", "v_mov_b64");
}
#undef MCRT_FLIGHT_ENTER
#undef MCRT_ENTER

#undef MCRT_DEP
#undef MCRT_CROSS_IN
#undef MCRT_CROSS_OUT
#undef MCRT_CROSS
#undef MCRT_AXIS_MASKS

}  // namespace mcrt
