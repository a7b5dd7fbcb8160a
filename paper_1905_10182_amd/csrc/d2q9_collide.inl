// The per-cell D2Q9 collision: included by d2q9.hpp, once per contraction mode
// and each time in a namespace of its own.

// inv1d with its first- and second-order inputs given at half scale
// (m1h = m1 / 2, m2h = m2 / 2) and hu = u / 2: with o = (g+ - g-) / 2 and
// e = (g+ + g-) / 2, o = m1h + hu m0, e = m2h + u (m1h + o), g-+ = e -+ o,
// g0 = m0 - 2 e.  Six operations instead of nine; the halving is folded into
// the construction of the moments (see reconstruct).
template <typename T>
__device__ __forceinline__ void inv1d_half(T m0, T m1h, T m2h, T u, T hu, T& gm, T& g0, T& gp)
{
    const T o = m1h + hu * m0;
    const T e = m2h + u * (m1h + o);
    gm = e - o;
    gp = e + o;
    g0 = m0 - T(2) * e;
}

// X = sum over cx of h (1, cx, cx^2) of one c_y class, given by c_x = -1, 0, +1.
template <typename T>
__device__ __forceinline__ void row_sums(T hm, T h0, T hp, T X[3])
{
    X[0] = hm + h0 + hp;
    X[1] = hp - hm;
    X[2] = hp + hm;
}

// Density deviation, half-force-corrected velocity and the two pre-collision
// central moments that relax with omega, k4 = sum f [(cx-ux)^2 - (cy-uy)^2]
// and k5 = sum f (cx-ux)(cy-uy), from the row sums of the c_y classes -1, 0,
// +1 of the pre-collision h.
template <typename T>
__device__ __forceinline__ void moments_of_sums(const T Xm[3], const T X0[3], const T Xp[3], T Fx, T Fy, T rho0,
                                                T& drho, T& ux, T& uy, T& k4, T& k5)
{
    drho = Xm[0] + X0[0] + Xp[0];
    const T jx = Xm[1] + X0[1] + Xp[1];
    const T jy = Xp[0] - Xm[0];
    const T Sxx = Xm[2] + X0[2] + Xp[2];
    const T Syy = Xp[0] + Xm[0];
    const T Sxy = Xp[1] - Xm[1];
    const T rho = rho0 + drho;
    const T inv_rho = T(1) / rho;
    ux = (jx + T(0.5) * Fx) * inv_rho;
    uy = (jy + T(0.5) * Fy) * inv_rho;
    // central from raw moments; the rest state adds nothing to Sxx - Syy or Sxy
    k4 = (Sxx - Syy) - rho * (ux * ux - uy * uy) + (ux * Fx - uy * Fy);
    k5 = Sxy - rho * ux * uy + T(0.5) * (ux * Fy + uy * Fx);
}

// The same from the nine populations of one cell.
template <typename T>
__device__ __forceinline__ void pre_collision(const T h[9], T Fx, T Fy, T rho0, T& drho, T& ux, T& uy, T& k4, T& k5)
{
    T X[3][3];
#pragma unroll
    for (int b = 0; b < 3; ++b)
        row_sums(h[vel_index(-1, b - 1)], h[vel_index(0, b - 1)], h[vel_index(1, b - 1)], X[b]);
    moments_of_sums(X[0], X[1], X[2], Fx, Fy, rho0, drho, ux, uy, k4, k5);
}

// Post-collision h*_i = f*_i - w_i rho0 from the density deviation, the
// velocity, the force density and the relaxed moments s4 = (1 - omega) k4,
// s5 = (1 - omega) k5: the printed post-collision central moments of App. B
// (k0* = rho, k1,2* = F/2, k3* = 2 rho cs^2, k4,5* = s4,5, k6* = Fy cs^2/2,
// k7* = Fx cs^2/2, k8* = rho cs^4) on the monomials (cx-ux)^p (cy-uy)^q, minus
// the rest-state moments rho0 M_p(ux) M_q(uy) (M_0 = 1, M_1(u) = -u,
// M_2(u) = 1/3 + u^2), then the inverse transform along y and along x.
// As in the D3Q27 reconstruction, D[p][q] is held at scale 2^-(number of
// non-zero p, q) so that both 1D passes take their first- and second-order
// inputs at half scale (inv1d_half); the populations come out unscaled.
template <typename T>
__device__ __forceinline__ void reconstruct(T drho, T ux, T uy, T Fx, T Fy, T s4, T s5, T rho0, T h[9])
{
    const T third = T(1.0 / 3.0);
    const T ux2 = ux * ux, uy2 = uy * uy;
    const T r1 = T(0.5) * rho0, r2 = T(0.25) * rho0;
    T D[3][3];
    D[0][0] = drho;
    D[1][0] = T(0.25) * Fx + r1 * ux;
    D[0][1] = T(0.25) * Fy + r1 * uy;
    D[2][0] = drho * T(1.0 / 6.0) + T(0.25) * s4 - r1 * ux2;
    D[0][2] = drho * T(1.0 / 6.0) - T(0.25) * s4 - r1 * uy2;
    D[1][1] = T(0.25) * s5 - r2 * ux * uy;
    D[2][1] = Fy * T(1.0 / 24.0) + r2 * uy * (third + ux2);
    D[1][2] = Fx * T(1.0 / 24.0) + r2 * ux * (third + uy2);
    D[2][2] = drho * T(1.0 / 36.0) - r2 * ((ux2 + uy2) * third + ux2 * uy2);
    const T hx = T(0.5) * ux, hy = T(0.5) * uy;
    T G[3][3];  // G[p][cy + 1]: x-moment p of the populations with that cy (at scale 2^-[p > 0])
#pragma unroll
    for (int p = 0; p < 3; ++p) inv1d_half<T>(D[p][0], D[p][1], D[p][2], uy, hy, G[p][0], G[p][1], G[p][2]);
#pragma unroll
    for (int b = 0; b < 3; ++b) {
        T gm, g0, gp;
        inv1d_half<T>(G[0][b], G[1][b], G[2][b], ux, hx, gm, g0, gp);
        h[vel_index(-1, b - 1)] = gm;
        h[vel_index(0, b - 1)] = g0;
        h[vel_index(1, b - 1)] = gp;
    }
}

// One collision in place: h (pre-collision) -> h* (post-collision); returns
// the density deviation and velocity of the cell.
template <typename T>
__device__ __forceinline__ void collide(T h[9], T Fx, T Fy, T omega, T rho0, T& drho, T& ux, T& uy)
{
    T k4, k5;
    pre_collision<T>(h, Fx, Fy, rho0, drho, ux, uy, k4, k5);
    const T r = T(1) - omega;
    reconstruct<T>(drho, ux, uy, Fx, Fy, r * k4, r * k5, rho0, h);
}
