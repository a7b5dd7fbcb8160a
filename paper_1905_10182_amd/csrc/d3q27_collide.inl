// The per-cell collision: included by d3q27.hpp, once per contraction mode and
// each time in a namespace of its own.

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

// In-plane sums of the nine populations of one c_z class, g[(cy + 1) * 3 + cx + 1]:
// Y = sum g * (1, cx, cy, cx^2, cy^2, cx cy), by 1D sums along x, then y.
template <typename T>
__device__ __forceinline__ void plane_sums(const T g[9], T Y[6])
{
    T X[3][3];  // X[p][b] = sum_a g(a, b) a^p
#pragma unroll
    for (int b = 0; b < 3; ++b) {
        X[0][b] = g[3 * b] + g[3 * b + 1] + g[3 * b + 2];
        X[1][b] = g[3 * b + 2] - g[3 * b];
        X[2][b] = g[3 * b + 2] + g[3 * b];
    }
    Y[0] = X[0][0] + X[0][1] + X[0][2];
    Y[1] = X[1][0] + X[1][1] + X[1][2];
    Y[2] = X[0][2] - X[0][0];
    Y[3] = X[2][0] + X[2][1] + X[2][2];
    Y[4] = X[0][2] + X[0][0];
    Y[5] = X[1][2] - X[1][0];
}

// First half of the collision: density, half-force-corrected velocity
// (eq. "macroscopic") and the five pre-collision central moments k4..k8
// (eq. "pre_collision") from the in-plane sums of the three c_z classes of
// the pre-collision h_i = f_i - w_i rho0.
template <typename T>
__device__ __forceinline__ void moments_of_sums(const T Ym[6], const T Y0[6], const T Yp[6], T Fx, T Fy, T Fz, T rho0,
                                                T& drho, T& ux, T& uy, T& uz, T k[5])
{
    drho = Ym[0] + Y0[0] + Yp[0];
    const T jx = Ym[1] + Y0[1] + Yp[1], jy = Ym[2] + Y0[2] + Yp[2], jz = Yp[0] - Ym[0];
    const T Sxx = Ym[3] + Y0[3] + Yp[3], Syy = Ym[4] + Y0[4] + Yp[4], Szz = Yp[0] + Ym[0];
    const T Sxy = Ym[5] + Y0[5] + Yp[5], Sxz = Yp[1] - Ym[1], Syz = Yp[2] - Ym[2];

    // Macroscopic variables with the half-force correction (eq. "macroscopic").
    const T rho = rho0 + drho;
    const T inv_rho = reciprocal(rho);
    ux = (jx + T(0.5) * Fx) * inv_rho;
    uy = (jy + T(0.5) * Fy) * inv_rho;
    uz = (jz + T(0.5) * Fz) * inv_rho;

    // The five pre-collision central moments k4..k8 from raw moments:
    // sum f (cx-ux)(cy-uy) = Pxy - rho ux uy + (ux Fy + uy Fx)/2, where the
    // rest state contributes nothing to Pxy or Pxx - Pyy.
    k[0] = Sxy - rho * ux * uy + T(0.5) * (ux * Fy + uy * Fx);
    k[1] = Sxz - rho * ux * uz + T(0.5) * (ux * Fz + uz * Fx);
    k[2] = Syz - rho * uy * uz + T(0.5) * (uy * Fz + uz * Fy);
    k[3] = (Sxx - Syy) - rho * (ux * ux - uy * uy) + (ux * Fx - uy * Fy);
    k[4] = (Sxx - Szz) - rho * (ux * ux - uz * uz) + (ux * Fx - uz * Fz);
}

// The same from the 27 populations of one cell.
template <typename T>
__device__ __forceinline__ void pre_collision(const T h[27], T Fx, T Fy, T Fz, T rho0, T& drho, T& ux, T& uy, T& uz,
                                              T k[5])
{
    T Y[3][6];
#pragma unroll
    for (int c = 0; c < 3; ++c) {
        T gz[9];
#pragma unroll
        for (int j = 0; j < 9; ++j) gz[j] = h[vel_index(j % 3 - 1, j / 3 - 1, c - 1)];
        plane_sums(gz, Y[c]);
    }
    moments_of_sums(Y[0], Y[1], Y[2], Fx, Fy, Fz, rho0, drho, ux, uy, uz, k);
}

// Second half: the post-collision populations h*_i = f*_i - w_i rho0 from
// the density deviation, the velocity, the force density and the relaxed
// shear moments s = (1 - omega) k4..k8, i.e. the nineteen non-zero
// post-collision central moments (eq. "post_collision_central_moments_forcing")
// and their inverse transform (eq. "system").
template <typename T>
__device__ __forceinline__ void reconstruct(T drho, T ux, T uy, T uz, T Fx, T Fy, T Fz, const T s[5], T rho0, T h[27])
{
    // Post-collision central moments on the monomials (cx-ux)^p (cy-uy)^q (cz-uz)^r,
    // minus the central moments of the rest state rho0 w_i, which factor as
    // rho0 M_p(ux) M_q(uy) M_r(uz) with M_0 = 1, M_1(u) = -u, M_2(u) = 1/3 + u^2.
    // D[p][q][r] is held at scale 2^-(number of non-zero p, q, r): each of the
    // three 1D passes below then receives its first- and second-order inputs
    // at half scale (inv1d_half), and by linearity the populations come out
    // unscaled.  The scale factors are powers of two, so they round nothing.
    const T third = T(1.0 / 3.0);
    const T ux2 = ux * ux, uy2 = uy * uy, uz2 = uz * uz;
    const T ax = third + ux2, ay = third + uy2, az = third + uz2;
    const T r1 = T(0.5) * rho0, r2 = T(0.25) * rho0, r3 = T(0.125) * rho0;
    T D[3][3][3];
    D[0][0][0] = drho;
    D[1][0][0] = T(0.25) * Fx + r1 * ux;
    D[0][1][0] = T(0.25) * Fy + r1 * uy;
    D[0][0][1] = T(0.25) * Fz + r1 * uz;
    D[1][1][0] = T(0.25) * s[0] - r2 * ux * uy;
    D[1][0][1] = T(0.25) * s[1] - r2 * ux * uz;
    D[0][1][1] = T(0.25) * s[2] - r2 * uy * uz;
    const T sixth = T(1.0 / 6.0);
    D[2][0][0] = (s[3] + s[4] + drho) * sixth - r1 * ux2;
    D[0][2][0] = (s[4] - T(2) * s[3] + drho) * sixth - r1 * uy2;
    D[0][0][2] = (s[3] - T(2) * s[4] + drho) * sixth - r1 * uz2;
    const T f24 = T(1.0 / 24.0);
    D[1][2][0] = f24 * Fx + r2 * ux * ay;
    D[1][0][2] = f24 * Fx + r2 * ux * az;
    D[2][1][0] = f24 * Fy + r2 * uy * ax;
    D[0][1][2] = f24 * Fy + r2 * uy * az;
    D[2][0][1] = f24 * Fz + r2 * uz * ax;
    D[0][2][1] = f24 * Fz + r2 * uz * ay;
    D[1][1][1] = r3 * ux * uy * uz;
    const T f36 = T(1.0 / 36.0);
    D[2][2][0] = f36 * drho - r2 * ((ux2 + uy2) * third + ux2 * uy2);
    D[2][0][2] = f36 * drho - r2 * ((ux2 + uz2) * third + ux2 * uz2);
    D[0][2][2] = f36 * drho - r2 * ((uy2 + uz2) * third + uy2 * uz2);
    D[2][1][1] = -r3 * ax * uy * uz;
    D[1][2][1] = -r3 * ay * ux * uz;
    D[1][1][2] = -r3 * az * ux * uy;
    const T f144 = T(1.0 / 144.0);
    D[1][2][2] = f144 * Fx + r3 * ux * ay * az;
    D[2][1][2] = f144 * Fy + r3 * uy * ax * az;
    D[2][2][1] = f144 * Fz + r3 * uz * ax * ay;
    D[2][2][2] = T(1.0 / 216.0) * drho -
                 r3 * ((ux2 + uy2 + uz2) * (T(1.0 / 9.0)) + (ux2 * uy2 + ux2 * uz2 + uy2 * uz2) * third + ux2 * uy2 * uz2);

    // Reconstruction (eq. "system") by the factorised inverse transform:
    // along z, then y, then x.
    const T hx = T(0.5) * ux, hy = T(0.5) * uy, hz = T(0.5) * uz;
    T A[3][3][3];
#pragma unroll
    for (int p = 0; p < 3; ++p)
#pragma unroll
        for (int q = 0; q < 3; ++q)
            inv1d_half(D[p][q][0], D[p][q][1], D[p][q][2], uz, hz, A[p][q][0], A[p][q][1], A[p][q][2]);
    T B[3][3][3];
#pragma unroll
    for (int p = 0; p < 3; ++p)
#pragma unroll
        for (int c = 0; c < 3; ++c)
            inv1d_half(A[p][0][c], A[p][1][c], A[p][2][c], uy, hy, B[p][0][c], B[p][1][c], B[p][2][c]);
#pragma unroll
    for (int b = 0; b < 3; ++b)
#pragma unroll
        for (int c = 0; c < 3; ++c)
            inv1d_half(B[0][b][c], B[1][b][c], B[2][b][c], ux, hx, h[vel_index(-1, b - 1, c - 1)],
                       h[vel_index(0, b - 1, c - 1)], h[vel_index(1, b - 1, c - 1)]);
}

// Collide one cell in place: pre-collision h_i in, post-collision h*_i out.
template <typename T>
__device__ __forceinline__ void collide(T h[27], T Fx, T Fy, T Fz, T omega, T rho0)
{
    T drho, ux, uy, uz, k[5], s[5];
    pre_collision(h, Fx, Fy, Fz, rho0, drho, ux, uy, uz, k);
    const T om1 = T(1) - omega;
#pragma unroll
    for (int j = 0; j < 5; ++j) s[j] = om1 * k[j];
    reconstruct(drho, ux, uy, uz, Fx, Fy, Fz, s, rho0, h);
}
