// Generated by gen_star_centre.py; do not edit.  The centre-row taps of a star footprint on N rows
// of V columns per lane at once (R <= V): o[n][c] += w[dx] * x[n][c + dx] for dx = -R..-1, then 1..R,
// in that order for every cell; columns beyond the lane are read from the neighbouring lanes by DPP
// operands, lanes at the wave's ends read 0.
#pragma once

namespace st {
namespace block {

template <int R, int V, int N>
struct StarRows {
    static constexpr bool exists = false;
};

template <>
struct StarRows<1, 1, 8> {
    static constexpr bool exists = true;
    __device__ __forceinline__ static void apply(float (*o)[1], const float (*x)[1], const float* w) {
        asm("s_nop 4\n"
        "v_fmac_f32_dpp %0, %8, %16 wave_shr:1 row_mask:0xf bank_mask:0xf bound_ctrl:1\n"
        "v_fmac_f32_dpp %1, %9, %16 wave_shr:1 row_mask:0xf bank_mask:0xf bound_ctrl:1\n"
        "v_fmac_f32_dpp %2, %10, %16 wave_shr:1 row_mask:0xf bank_mask:0xf bound_ctrl:1\n"
        "v_fmac_f32_dpp %3, %11, %16 wave_shr:1 row_mask:0xf bank_mask:0xf bound_ctrl:1\n"
        "v_fmac_f32_dpp %4, %12, %16 wave_shr:1 row_mask:0xf bank_mask:0xf bound_ctrl:1\n"
        "v_fmac_f32_dpp %5, %13, %16 wave_shr:1 row_mask:0xf bank_mask:0xf bound_ctrl:1\n"
        "v_fmac_f32_dpp %6, %14, %16 wave_shr:1 row_mask:0xf bank_mask:0xf bound_ctrl:1\n"
        "v_fmac_f32_dpp %7, %15, %16 wave_shr:1 row_mask:0xf bank_mask:0xf bound_ctrl:1\n"
        "v_fmac_f32_dpp %0, %8, %17 wave_shl:1 row_mask:0xf bank_mask:0xf bound_ctrl:1\n"
        "v_fmac_f32_dpp %1, %9, %17 wave_shl:1 row_mask:0xf bank_mask:0xf bound_ctrl:1\n"
        "v_fmac_f32_dpp %2, %10, %17 wave_shl:1 row_mask:0xf bank_mask:0xf bound_ctrl:1\n"
        "v_fmac_f32_dpp %3, %11, %17 wave_shl:1 row_mask:0xf bank_mask:0xf bound_ctrl:1\n"
        "v_fmac_f32_dpp %4, %12, %17 wave_shl:1 row_mask:0xf bank_mask:0xf bound_ctrl:1\n"
        "v_fmac_f32_dpp %5, %13, %17 wave_shl:1 row_mask:0xf bank_mask:0xf bound_ctrl:1\n"
        "v_fmac_f32_dpp %6, %14, %17 wave_shl:1 row_mask:0xf bank_mask:0xf bound_ctrl:1\n"
        "v_fmac_f32_dpp %7, %15, %17 wave_shl:1 row_mask:0xf bank_mask:0xf bound_ctrl:1"
            : "+v"(o[0][0]), "+v"(o[1][0]), "+v"(o[2][0]), "+v"(o[3][0]), "+v"(o[4][0]), "+v"(o[5][0]), "+v"(o[6][0]), "+v"(o[7][0])
            : "v"(x[0][0]), "v"(x[1][0]), "v"(x[2][0]), "v"(x[3][0]), "v"(x[4][0]), "v"(x[5][0]), "v"(x[6][0]), "v"(x[7][0]), "v"(w[0]), "v"(w[1]));
    }
};

template <>
struct StarRows<1, 1, 4> {
    static constexpr bool exists = true;
    __device__ __forceinline__ static void apply(float (*o)[1], const float (*x)[1], const float* w) {
        asm("s_nop 4\n"
        "v_fmac_f32_dpp %0, %4, %8 wave_shr:1 row_mask:0xf bank_mask:0xf bound_ctrl:1\n"
        "v_fmac_f32_dpp %1, %5, %8 wave_shr:1 row_mask:0xf bank_mask:0xf bound_ctrl:1\n"
        "v_fmac_f32_dpp %2, %6, %8 wave_shr:1 row_mask:0xf bank_mask:0xf bound_ctrl:1\n"
        "v_fmac_f32_dpp %3, %7, %8 wave_shr:1 row_mask:0xf bank_mask:0xf bound_ctrl:1\n"
        "v_fmac_f32_dpp %0, %4, %9 wave_shl:1 row_mask:0xf bank_mask:0xf bound_ctrl:1\n"
        "v_fmac_f32_dpp %1, %5, %9 wave_shl:1 row_mask:0xf bank_mask:0xf bound_ctrl:1\n"
        "v_fmac_f32_dpp %2, %6, %9 wave_shl:1 row_mask:0xf bank_mask:0xf bound_ctrl:1\n"
        "v_fmac_f32_dpp %3, %7, %9 wave_shl:1 row_mask:0xf bank_mask:0xf bound_ctrl:1"
            : "+v"(o[0][0]), "+v"(o[1][0]), "+v"(o[2][0]), "+v"(o[3][0])
            : "v"(x[0][0]), "v"(x[1][0]), "v"(x[2][0]), "v"(x[3][0]), "v"(w[0]), "v"(w[1]));
    }
};

template <>
struct StarRows<1, 2, 4> {
    static constexpr bool exists = true;
    __device__ __forceinline__ static void apply(float (*o)[2], const float (*x)[2], const float* w) {
        asm("s_nop 4\n"
        "v_fmac_f32_dpp %0, %9, %16 wave_shr:1 row_mask:0xf bank_mask:0xf bound_ctrl:1\n"
        "v_fmac_f32_e32 %1, %8, %16\n"
        "v_fmac_f32_dpp %2, %11, %16 wave_shr:1 row_mask:0xf bank_mask:0xf bound_ctrl:1\n"
        "v_fmac_f32_e32 %3, %10, %16\n"
        "v_fmac_f32_dpp %4, %13, %16 wave_shr:1 row_mask:0xf bank_mask:0xf bound_ctrl:1\n"
        "v_fmac_f32_e32 %5, %12, %16\n"
        "v_fmac_f32_dpp %6, %15, %16 wave_shr:1 row_mask:0xf bank_mask:0xf bound_ctrl:1\n"
        "v_fmac_f32_e32 %7, %14, %16\n"
        "v_fmac_f32_e32 %0, %9, %17\n"
        "v_fmac_f32_dpp %1, %8, %17 wave_shl:1 row_mask:0xf bank_mask:0xf bound_ctrl:1\n"
        "v_fmac_f32_e32 %2, %11, %17\n"
        "v_fmac_f32_dpp %3, %10, %17 wave_shl:1 row_mask:0xf bank_mask:0xf bound_ctrl:1\n"
        "v_fmac_f32_e32 %4, %13, %17\n"
        "v_fmac_f32_dpp %5, %12, %17 wave_shl:1 row_mask:0xf bank_mask:0xf bound_ctrl:1\n"
        "v_fmac_f32_e32 %6, %15, %17\n"
        "v_fmac_f32_dpp %7, %14, %17 wave_shl:1 row_mask:0xf bank_mask:0xf bound_ctrl:1"
            : "+v"(o[0][0]), "+v"(o[0][1]), "+v"(o[1][0]), "+v"(o[1][1]), "+v"(o[2][0]), "+v"(o[2][1]), "+v"(o[3][0]), "+v"(o[3][1])
            : "v"(x[0][0]), "v"(x[0][1]), "v"(x[1][0]), "v"(x[1][1]), "v"(x[2][0]), "v"(x[2][1]), "v"(x[3][0]), "v"(x[3][1]), "v"(w[0]), "v"(w[1]));
    }
};

template <>
struct StarRows<2, 2, 4> {
    static constexpr bool exists = true;
    __device__ __forceinline__ static void apply(float (*o)[2], const float (*x)[2], const float* w) {
        asm("s_nop 4\n"
        "v_fmac_f32_dpp %0, %8, %16 wave_shr:1 row_mask:0xf bank_mask:0xf bound_ctrl:1\n"
        "v_fmac_f32_dpp %1, %9, %16 wave_shr:1 row_mask:0xf bank_mask:0xf bound_ctrl:1\n"
        "v_fmac_f32_dpp %2, %10, %16 wave_shr:1 row_mask:0xf bank_mask:0xf bound_ctrl:1\n"
        "v_fmac_f32_dpp %3, %11, %16 wave_shr:1 row_mask:0xf bank_mask:0xf bound_ctrl:1\n"
        "v_fmac_f32_dpp %4, %12, %16 wave_shr:1 row_mask:0xf bank_mask:0xf bound_ctrl:1\n"
        "v_fmac_f32_dpp %5, %13, %16 wave_shr:1 row_mask:0xf bank_mask:0xf bound_ctrl:1\n"
        "v_fmac_f32_dpp %6, %14, %16 wave_shr:1 row_mask:0xf bank_mask:0xf bound_ctrl:1\n"
        "v_fmac_f32_dpp %7, %15, %16 wave_shr:1 row_mask:0xf bank_mask:0xf bound_ctrl:1\n"
        "v_fmac_f32_dpp %0, %9, %17 wave_shr:1 row_mask:0xf bank_mask:0xf bound_ctrl:1\n"
        "v_fmac_f32_e32 %1, %8, %17\n"
        "v_fmac_f32_dpp %2, %11, %17 wave_shr:1 row_mask:0xf bank_mask:0xf bound_ctrl:1\n"
        "v_fmac_f32_e32 %3, %10, %17\n"
        "v_fmac_f32_dpp %4, %13, %17 wave_shr:1 row_mask:0xf bank_mask:0xf bound_ctrl:1\n"
        "v_fmac_f32_e32 %5, %12, %17\n"
        "v_fmac_f32_dpp %6, %15, %17 wave_shr:1 row_mask:0xf bank_mask:0xf bound_ctrl:1\n"
        "v_fmac_f32_e32 %7, %14, %17\n"
        "v_fmac_f32_e32 %0, %9, %18\n"
        "v_fmac_f32_dpp %1, %8, %18 wave_shl:1 row_mask:0xf bank_mask:0xf bound_ctrl:1\n"
        "v_fmac_f32_e32 %2, %11, %18\n"
        "v_fmac_f32_dpp %3, %10, %18 wave_shl:1 row_mask:0xf bank_mask:0xf bound_ctrl:1\n"
        "v_fmac_f32_e32 %4, %13, %18\n"
        "v_fmac_f32_dpp %5, %12, %18 wave_shl:1 row_mask:0xf bank_mask:0xf bound_ctrl:1\n"
        "v_fmac_f32_e32 %6, %15, %18\n"
        "v_fmac_f32_dpp %7, %14, %18 wave_shl:1 row_mask:0xf bank_mask:0xf bound_ctrl:1\n"
        "v_fmac_f32_dpp %0, %8, %19 wave_shl:1 row_mask:0xf bank_mask:0xf bound_ctrl:1\n"
        "v_fmac_f32_dpp %1, %9, %19 wave_shl:1 row_mask:0xf bank_mask:0xf bound_ctrl:1\n"
        "v_fmac_f32_dpp %2, %10, %19 wave_shl:1 row_mask:0xf bank_mask:0xf bound_ctrl:1\n"
        "v_fmac_f32_dpp %3, %11, %19 wave_shl:1 row_mask:0xf bank_mask:0xf bound_ctrl:1\n"
        "v_fmac_f32_dpp %4, %12, %19 wave_shl:1 row_mask:0xf bank_mask:0xf bound_ctrl:1\n"
        "v_fmac_f32_dpp %5, %13, %19 wave_shl:1 row_mask:0xf bank_mask:0xf bound_ctrl:1\n"
        "v_fmac_f32_dpp %6, %14, %19 wave_shl:1 row_mask:0xf bank_mask:0xf bound_ctrl:1\n"
        "v_fmac_f32_dpp %7, %15, %19 wave_shl:1 row_mask:0xf bank_mask:0xf bound_ctrl:1"
            : "+v"(o[0][0]), "+v"(o[0][1]), "+v"(o[1][0]), "+v"(o[1][1]), "+v"(o[2][0]), "+v"(o[2][1]), "+v"(o[3][0]), "+v"(o[3][1])
            : "v"(x[0][0]), "v"(x[0][1]), "v"(x[1][0]), "v"(x[1][1]), "v"(x[2][0]), "v"(x[2][1]), "v"(x[3][0]), "v"(x[3][1]), "v"(w[0]), "v"(w[1]), "v"(w[2]), "v"(w[3]));
    }
};

template <>
struct StarRows<1, 4, 2> {
    static constexpr bool exists = true;
    __device__ __forceinline__ static void apply(float (*o)[4], const float (*x)[4], const float* w) {
        asm("s_nop 4\n"
        "v_fmac_f32_dpp %0, %11, %16 wave_shr:1 row_mask:0xf bank_mask:0xf bound_ctrl:1\n"
        "v_fmac_f32_e32 %1, %8, %16\n"
        "v_fmac_f32_e32 %2, %9, %16\n"
        "v_fmac_f32_e32 %3, %10, %16\n"
        "v_fmac_f32_dpp %4, %15, %16 wave_shr:1 row_mask:0xf bank_mask:0xf bound_ctrl:1\n"
        "v_fmac_f32_e32 %5, %12, %16\n"
        "v_fmac_f32_e32 %6, %13, %16\n"
        "v_fmac_f32_e32 %7, %14, %16\n"
        "v_fmac_f32_e32 %0, %9, %17\n"
        "v_fmac_f32_e32 %1, %10, %17\n"
        "v_fmac_f32_e32 %2, %11, %17\n"
        "v_fmac_f32_dpp %3, %8, %17 wave_shl:1 row_mask:0xf bank_mask:0xf bound_ctrl:1\n"
        "v_fmac_f32_e32 %4, %13, %17\n"
        "v_fmac_f32_e32 %5, %14, %17\n"
        "v_fmac_f32_e32 %6, %15, %17\n"
        "v_fmac_f32_dpp %7, %12, %17 wave_shl:1 row_mask:0xf bank_mask:0xf bound_ctrl:1"
            : "+v"(o[0][0]), "+v"(o[0][1]), "+v"(o[0][2]), "+v"(o[0][3]), "+v"(o[1][0]), "+v"(o[1][1]), "+v"(o[1][2]), "+v"(o[1][3])
            : "v"(x[0][0]), "v"(x[0][1]), "v"(x[0][2]), "v"(x[0][3]), "v"(x[1][0]), "v"(x[1][1]), "v"(x[1][2]), "v"(x[1][3]), "v"(w[0]), "v"(w[1]));
    }
};

template <>
struct StarRows<2, 4, 2> {
    static constexpr bool exists = true;
    __device__ __forceinline__ static void apply(float (*o)[4], const float (*x)[4], const float* w) {
        asm("s_nop 4\n"
        "v_fmac_f32_dpp %0, %10, %16 wave_shr:1 row_mask:0xf bank_mask:0xf bound_ctrl:1\n"
        "v_fmac_f32_dpp %1, %11, %16 wave_shr:1 row_mask:0xf bank_mask:0xf bound_ctrl:1\n"
        "v_fmac_f32_e32 %2, %8, %16\n"
        "v_fmac_f32_e32 %3, %9, %16\n"
        "v_fmac_f32_dpp %4, %14, %16 wave_shr:1 row_mask:0xf bank_mask:0xf bound_ctrl:1\n"
        "v_fmac_f32_dpp %5, %15, %16 wave_shr:1 row_mask:0xf bank_mask:0xf bound_ctrl:1\n"
        "v_fmac_f32_e32 %6, %12, %16\n"
        "v_fmac_f32_e32 %7, %13, %16\n"
        "v_fmac_f32_dpp %0, %11, %17 wave_shr:1 row_mask:0xf bank_mask:0xf bound_ctrl:1\n"
        "v_fmac_f32_e32 %1, %8, %17\n"
        "v_fmac_f32_e32 %2, %9, %17\n"
        "v_fmac_f32_e32 %3, %10, %17\n"
        "v_fmac_f32_dpp %4, %15, %17 wave_shr:1 row_mask:0xf bank_mask:0xf bound_ctrl:1\n"
        "v_fmac_f32_e32 %5, %12, %17\n"
        "v_fmac_f32_e32 %6, %13, %17\n"
        "v_fmac_f32_e32 %7, %14, %17\n"
        "v_fmac_f32_e32 %0, %9, %18\n"
        "v_fmac_f32_e32 %1, %10, %18\n"
        "v_fmac_f32_e32 %2, %11, %18\n"
        "v_fmac_f32_dpp %3, %8, %18 wave_shl:1 row_mask:0xf bank_mask:0xf bound_ctrl:1\n"
        "v_fmac_f32_e32 %4, %13, %18\n"
        "v_fmac_f32_e32 %5, %14, %18\n"
        "v_fmac_f32_e32 %6, %15, %18\n"
        "v_fmac_f32_dpp %7, %12, %18 wave_shl:1 row_mask:0xf bank_mask:0xf bound_ctrl:1\n"
        "v_fmac_f32_e32 %0, %10, %19\n"
        "v_fmac_f32_e32 %1, %11, %19\n"
        "v_fmac_f32_dpp %2, %8, %19 wave_shl:1 row_mask:0xf bank_mask:0xf bound_ctrl:1\n"
        "v_fmac_f32_dpp %3, %9, %19 wave_shl:1 row_mask:0xf bank_mask:0xf bound_ctrl:1\n"
        "v_fmac_f32_e32 %4, %14, %19\n"
        "v_fmac_f32_e32 %5, %15, %19\n"
        "v_fmac_f32_dpp %6, %12, %19 wave_shl:1 row_mask:0xf bank_mask:0xf bound_ctrl:1\n"
        "v_fmac_f32_dpp %7, %13, %19 wave_shl:1 row_mask:0xf bank_mask:0xf bound_ctrl:1"
            : "+v"(o[0][0]), "+v"(o[0][1]), "+v"(o[0][2]), "+v"(o[0][3]), "+v"(o[1][0]), "+v"(o[1][1]), "+v"(o[1][2]), "+v"(o[1][3])
            : "v"(x[0][0]), "v"(x[0][1]), "v"(x[0][2]), "v"(x[0][3]), "v"(x[1][0]), "v"(x[1][1]), "v"(x[1][2]), "v"(x[1][3]), "v"(w[0]), "v"(w[1]), "v"(w[2]), "v"(w[3]));
    }
};

template <>
struct StarRows<3, 4, 2> {
    static constexpr bool exists = true;
    __device__ __forceinline__ static void apply(float (*o)[4], const float (*x)[4], const float* w) {
        asm("s_nop 4\n"
        "v_fmac_f32_dpp %0, %9, %16 wave_shr:1 row_mask:0xf bank_mask:0xf bound_ctrl:1\n"
        "v_fmac_f32_dpp %1, %10, %16 wave_shr:1 row_mask:0xf bank_mask:0xf bound_ctrl:1\n"
        "v_fmac_f32_dpp %2, %11, %16 wave_shr:1 row_mask:0xf bank_mask:0xf bound_ctrl:1\n"
        "v_fmac_f32_e32 %3, %8, %16\n"
        "v_fmac_f32_dpp %4, %13, %16 wave_shr:1 row_mask:0xf bank_mask:0xf bound_ctrl:1\n"
        "v_fmac_f32_dpp %5, %14, %16 wave_shr:1 row_mask:0xf bank_mask:0xf bound_ctrl:1\n"
        "v_fmac_f32_dpp %6, %15, %16 wave_shr:1 row_mask:0xf bank_mask:0xf bound_ctrl:1\n"
        "v_fmac_f32_e32 %7, %12, %16\n"
        "v_fmac_f32_dpp %0, %10, %17 wave_shr:1 row_mask:0xf bank_mask:0xf bound_ctrl:1\n"
        "v_fmac_f32_dpp %1, %11, %17 wave_shr:1 row_mask:0xf bank_mask:0xf bound_ctrl:1\n"
        "v_fmac_f32_e32 %2, %8, %17\n"
        "v_fmac_f32_e32 %3, %9, %17\n"
        "v_fmac_f32_dpp %4, %14, %17 wave_shr:1 row_mask:0xf bank_mask:0xf bound_ctrl:1\n"
        "v_fmac_f32_dpp %5, %15, %17 wave_shr:1 row_mask:0xf bank_mask:0xf bound_ctrl:1\n"
        "v_fmac_f32_e32 %6, %12, %17\n"
        "v_fmac_f32_e32 %7, %13, %17\n"
        "v_fmac_f32_dpp %0, %11, %18 wave_shr:1 row_mask:0xf bank_mask:0xf bound_ctrl:1\n"
        "v_fmac_f32_e32 %1, %8, %18\n"
        "v_fmac_f32_e32 %2, %9, %18\n"
        "v_fmac_f32_e32 %3, %10, %18\n"
        "v_fmac_f32_dpp %4, %15, %18 wave_shr:1 row_mask:0xf bank_mask:0xf bound_ctrl:1\n"
        "v_fmac_f32_e32 %5, %12, %18\n"
        "v_fmac_f32_e32 %6, %13, %18\n"
        "v_fmac_f32_e32 %7, %14, %18\n"
        "v_fmac_f32_e32 %0, %9, %19\n"
        "v_fmac_f32_e32 %1, %10, %19\n"
        "v_fmac_f32_e32 %2, %11, %19\n"
        "v_fmac_f32_dpp %3, %8, %19 wave_shl:1 row_mask:0xf bank_mask:0xf bound_ctrl:1\n"
        "v_fmac_f32_e32 %4, %13, %19\n"
        "v_fmac_f32_e32 %5, %14, %19\n"
        "v_fmac_f32_e32 %6, %15, %19\n"
        "v_fmac_f32_dpp %7, %12, %19 wave_shl:1 row_mask:0xf bank_mask:0xf bound_ctrl:1\n"
        "v_fmac_f32_e32 %0, %10, %20\n"
        "v_fmac_f32_e32 %1, %11, %20\n"
        "v_fmac_f32_dpp %2, %8, %20 wave_shl:1 row_mask:0xf bank_mask:0xf bound_ctrl:1\n"
        "v_fmac_f32_dpp %3, %9, %20 wave_shl:1 row_mask:0xf bank_mask:0xf bound_ctrl:1\n"
        "v_fmac_f32_e32 %4, %14, %20\n"
        "v_fmac_f32_e32 %5, %15, %20\n"
        "v_fmac_f32_dpp %6, %12, %20 wave_shl:1 row_mask:0xf bank_mask:0xf bound_ctrl:1\n"
        "v_fmac_f32_dpp %7, %13, %20 wave_shl:1 row_mask:0xf bank_mask:0xf bound_ctrl:1\n"
        "v_fmac_f32_e32 %0, %11, %21\n"
        "v_fmac_f32_dpp %1, %8, %21 wave_shl:1 row_mask:0xf bank_mask:0xf bound_ctrl:1\n"
        "v_fmac_f32_dpp %2, %9, %21 wave_shl:1 row_mask:0xf bank_mask:0xf bound_ctrl:1\n"
        "v_fmac_f32_dpp %3, %10, %21 wave_shl:1 row_mask:0xf bank_mask:0xf bound_ctrl:1\n"
        "v_fmac_f32_e32 %4, %15, %21\n"
        "v_fmac_f32_dpp %5, %12, %21 wave_shl:1 row_mask:0xf bank_mask:0xf bound_ctrl:1\n"
        "v_fmac_f32_dpp %6, %13, %21 wave_shl:1 row_mask:0xf bank_mask:0xf bound_ctrl:1\n"
        "v_fmac_f32_dpp %7, %14, %21 wave_shl:1 row_mask:0xf bank_mask:0xf bound_ctrl:1"
            : "+v"(o[0][0]), "+v"(o[0][1]), "+v"(o[0][2]), "+v"(o[0][3]), "+v"(o[1][0]), "+v"(o[1][1]), "+v"(o[1][2]), "+v"(o[1][3])
            : "v"(x[0][0]), "v"(x[0][1]), "v"(x[0][2]), "v"(x[0][3]), "v"(x[1][0]), "v"(x[1][1]), "v"(x[1][2]), "v"(x[1][3]), "v"(w[0]), "v"(w[1]), "v"(w[2]), "v"(w[3]), "v"(w[4]), "v"(w[5]));
    }
};

template <>
struct StarRows<4, 4, 2> {
    static constexpr bool exists = true;
    __device__ __forceinline__ static void apply(float (*o)[4], const float (*x)[4], const float* w) {
        asm("s_nop 4\n"
        "v_fmac_f32_dpp %0, %8, %16 wave_shr:1 row_mask:0xf bank_mask:0xf bound_ctrl:1\n"
        "v_fmac_f32_dpp %1, %9, %16 wave_shr:1 row_mask:0xf bank_mask:0xf bound_ctrl:1\n"
        "v_fmac_f32_dpp %2, %10, %16 wave_shr:1 row_mask:0xf bank_mask:0xf bound_ctrl:1\n"
        "v_fmac_f32_dpp %3, %11, %16 wave_shr:1 row_mask:0xf bank_mask:0xf bound_ctrl:1\n"
        "v_fmac_f32_dpp %4, %12, %16 wave_shr:1 row_mask:0xf bank_mask:0xf bound_ctrl:1\n"
        "v_fmac_f32_dpp %5, %13, %16 wave_shr:1 row_mask:0xf bank_mask:0xf bound_ctrl:1\n"
        "v_fmac_f32_dpp %6, %14, %16 wave_shr:1 row_mask:0xf bank_mask:0xf bound_ctrl:1\n"
        "v_fmac_f32_dpp %7, %15, %16 wave_shr:1 row_mask:0xf bank_mask:0xf bound_ctrl:1\n"
        "v_fmac_f32_dpp %0, %9, %17 wave_shr:1 row_mask:0xf bank_mask:0xf bound_ctrl:1\n"
        "v_fmac_f32_dpp %1, %10, %17 wave_shr:1 row_mask:0xf bank_mask:0xf bound_ctrl:1\n"
        "v_fmac_f32_dpp %2, %11, %17 wave_shr:1 row_mask:0xf bank_mask:0xf bound_ctrl:1\n"
        "v_fmac_f32_e32 %3, %8, %17\n"
        "v_fmac_f32_dpp %4, %13, %17 wave_shr:1 row_mask:0xf bank_mask:0xf bound_ctrl:1\n"
        "v_fmac_f32_dpp %5, %14, %17 wave_shr:1 row_mask:0xf bank_mask:0xf bound_ctrl:1\n"
        "v_fmac_f32_dpp %6, %15, %17 wave_shr:1 row_mask:0xf bank_mask:0xf bound_ctrl:1\n"
        "v_fmac_f32_e32 %7, %12, %17\n"
        "v_fmac_f32_dpp %0, %10, %18 wave_shr:1 row_mask:0xf bank_mask:0xf bound_ctrl:1\n"
        "v_fmac_f32_dpp %1, %11, %18 wave_shr:1 row_mask:0xf bank_mask:0xf bound_ctrl:1\n"
        "v_fmac_f32_e32 %2, %8, %18\n"
        "v_fmac_f32_e32 %3, %9, %18\n"
        "v_fmac_f32_dpp %4, %14, %18 wave_shr:1 row_mask:0xf bank_mask:0xf bound_ctrl:1\n"
        "v_fmac_f32_dpp %5, %15, %18 wave_shr:1 row_mask:0xf bank_mask:0xf bound_ctrl:1\n"
        "v_fmac_f32_e32 %6, %12, %18\n"
        "v_fmac_f32_e32 %7, %13, %18\n"
        "v_fmac_f32_dpp %0, %11, %19 wave_shr:1 row_mask:0xf bank_mask:0xf bound_ctrl:1\n"
        "v_fmac_f32_e32 %1, %8, %19\n"
        "v_fmac_f32_e32 %2, %9, %19\n"
        "v_fmac_f32_e32 %3, %10, %19\n"
        "v_fmac_f32_dpp %4, %15, %19 wave_shr:1 row_mask:0xf bank_mask:0xf bound_ctrl:1\n"
        "v_fmac_f32_e32 %5, %12, %19\n"
        "v_fmac_f32_e32 %6, %13, %19\n"
        "v_fmac_f32_e32 %7, %14, %19\n"
        "v_fmac_f32_e32 %0, %9, %20\n"
        "v_fmac_f32_e32 %1, %10, %20\n"
        "v_fmac_f32_e32 %2, %11, %20\n"
        "v_fmac_f32_dpp %3, %8, %20 wave_shl:1 row_mask:0xf bank_mask:0xf bound_ctrl:1\n"
        "v_fmac_f32_e32 %4, %13, %20\n"
        "v_fmac_f32_e32 %5, %14, %20\n"
        "v_fmac_f32_e32 %6, %15, %20\n"
        "v_fmac_f32_dpp %7, %12, %20 wave_shl:1 row_mask:0xf bank_mask:0xf bound_ctrl:1\n"
        "v_fmac_f32_e32 %0, %10, %21\n"
        "v_fmac_f32_e32 %1, %11, %21\n"
        "v_fmac_f32_dpp %2, %8, %21 wave_shl:1 row_mask:0xf bank_mask:0xf bound_ctrl:1\n"
        "v_fmac_f32_dpp %3, %9, %21 wave_shl:1 row_mask:0xf bank_mask:0xf bound_ctrl:1\n"
        "v_fmac_f32_e32 %4, %14, %21\n"
        "v_fmac_f32_e32 %5, %15, %21\n"
        "v_fmac_f32_dpp %6, %12, %21 wave_shl:1 row_mask:0xf bank_mask:0xf bound_ctrl:1\n"
        "v_fmac_f32_dpp %7, %13, %21 wave_shl:1 row_mask:0xf bank_mask:0xf bound_ctrl:1\n"
        "v_fmac_f32_e32 %0, %11, %22\n"
        "v_fmac_f32_dpp %1, %8, %22 wave_shl:1 row_mask:0xf bank_mask:0xf bound_ctrl:1\n"
        "v_fmac_f32_dpp %2, %9, %22 wave_shl:1 row_mask:0xf bank_mask:0xf bound_ctrl:1\n"
        "v_fmac_f32_dpp %3, %10, %22 wave_shl:1 row_mask:0xf bank_mask:0xf bound_ctrl:1\n"
        "v_fmac_f32_e32 %4, %15, %22\n"
        "v_fmac_f32_dpp %5, %12, %22 wave_shl:1 row_mask:0xf bank_mask:0xf bound_ctrl:1\n"
        "v_fmac_f32_dpp %6, %13, %22 wave_shl:1 row_mask:0xf bank_mask:0xf bound_ctrl:1\n"
        "v_fmac_f32_dpp %7, %14, %22 wave_shl:1 row_mask:0xf bank_mask:0xf bound_ctrl:1\n"
        "v_fmac_f32_dpp %0, %8, %23 wave_shl:1 row_mask:0xf bank_mask:0xf bound_ctrl:1\n"
        "v_fmac_f32_dpp %1, %9, %23 wave_shl:1 row_mask:0xf bank_mask:0xf bound_ctrl:1\n"
        "v_fmac_f32_dpp %2, %10, %23 wave_shl:1 row_mask:0xf bank_mask:0xf bound_ctrl:1\n"
        "v_fmac_f32_dpp %3, %11, %23 wave_shl:1 row_mask:0xf bank_mask:0xf bound_ctrl:1\n"
        "v_fmac_f32_dpp %4, %12, %23 wave_shl:1 row_mask:0xf bank_mask:0xf bound_ctrl:1\n"
        "v_fmac_f32_dpp %5, %13, %23 wave_shl:1 row_mask:0xf bank_mask:0xf bound_ctrl:1\n"
        "v_fmac_f32_dpp %6, %14, %23 wave_shl:1 row_mask:0xf bank_mask:0xf bound_ctrl:1\n"
        "v_fmac_f32_dpp %7, %15, %23 wave_shl:1 row_mask:0xf bank_mask:0xf bound_ctrl:1"
            : "+v"(o[0][0]), "+v"(o[0][1]), "+v"(o[0][2]), "+v"(o[0][3]), "+v"(o[1][0]), "+v"(o[1][1]), "+v"(o[1][2]), "+v"(o[1][3])
            : "v"(x[0][0]), "v"(x[0][1]), "v"(x[0][2]), "v"(x[0][3]), "v"(x[1][0]), "v"(x[1][1]), "v"(x[1][2]), "v"(x[1][3]), "v"(w[0]), "v"(w[1]), "v"(w[2]), "v"(w[3]), "v"(w[4]), "v"(w[5]), "v"(w[6]), "v"(w[7]));
    }
};

}  // namespace block
}  // namespace st
