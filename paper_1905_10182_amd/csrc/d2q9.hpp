// D2Q9 lattice constants and the per-cell collision of the two-dimensional
// central-moment lattice Boltzmann model with Hermite forcing (De Rosis, Huang
// & Coreixas, PRE 2019, App. B), for register-resident evaluation on gfx950.
//
// Deviation form, as in the three-dimensional solver: populations are handled
// as h_i = f_i - w_i rho0 and every central moment is carried minus its value
// for the rest state, so FP32 keeps its relative precision on the small
// quantities that carry the flow.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace cmlbm2d {

// Velocity components in the order of App. B.
__host__ __device__ constexpr int vel_x(int i)
{
    constexpr int v[9] = {0, 1, -1, 0, 0, 1, -1, 1, -1};
    return v[i];
}
__host__ __device__ constexpr int vel_y(int i)
{
    constexpr int v[9] = {0, 0, 0, 1, -1, 1, -1, -1, 1};
    return v[i];
}
// Index of the velocity (a, b), each in {-1, 0, 1}.
__host__ __device__ constexpr int vel_index(int a, int b)
{
    for (int i = 0; i < 9; ++i)
        if (vel_x(i) == a && vel_y(i) == b) return i;
    return -1;
}
// Lattice weight: the product of the 1D weights (1/6, 2/3, 1/6), i.e. 4/9,
// 1/9, 1/36 for |c|^2 = 0, 1, 2.
__host__ __device__ constexpr double weight(int i)
{
    return (vel_x(i) ? 1.0 / 6.0 : 2.0 / 3.0) * (vel_y(i) ? 1.0 / 6.0 : 2.0 / 3.0);
}

// The collision, compiled twice with one difference: where the compiler may
// join a multiplication and an addition into one rounding.
//   lockstep  only within one source expression (contract(on)): the same
//             numbers in every kernel that inlines it.  FP64 and FP32 storage,
//             whose steps run in k2_step or several at a time in k2_march, so
//             that any split of a run into calls gives the same bits.
//   joined    anywhere (the HIP default, contract(fast)): 16-bit storage,
//             which has one step kernel.
namespace lockstep {
#pragma clang fp contract(on)
#include "d2q9_collide.inl"
}  // namespace lockstep
namespace joined {
#pragma clang fp contract(fast)
#include "d2q9_collide.inl"
}  // namespace joined

}  // namespace cmlbm2d
