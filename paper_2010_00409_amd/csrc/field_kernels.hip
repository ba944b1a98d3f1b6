// Pulse initialisation with mapping into the periodic layer, focal-window
// cut-out and deterministic reductions.  Built with -ffp-contract=off so the
// float64 geometry (radii, angles, cut-out decisions) rounds like a plain
// evaluation of the same expressions.
#include "kernels.h"

namespace tf {

// ---------------------------------------------------------------- profiles
// Transverse profile: flat-top of Eq. (5) (first window half-open) or the
// Gaussian exp(-a^2/theta^2) of Sec. III.B.1 restricted to a <= pi/2.
__device__ double u_ts(double alpha, const PulseDev& p) {
    if (p.transverse == 0) {
        const double lo = p.theta - 0.5 * p.eps, hi = p.theta + 0.5 * p.eps;
        if (alpha < lo) return 1.0;
        if (alpha <= hi) {
            const double c = cos(M_PI * (alpha - p.theta + 0.5 * p.eps) / (2.0 * p.eps));
            return c * c;
        }
        return 0.0;
    }
    if (alpha <= 0.5 * M_PI) return exp(-(alpha * alpha) / (p.theta * p.theta));
    return 0.0;
}

// Longitudinal profile with carrier, zeta inside [-L/2, L/2] (checked by the
// caller), for the cos^2 envelope of Eq. (7) and the Gaussian envelope of
// Sec. III.B.1.
template <int ENV> __device__ __forceinline__ double u_l_closed(double zeta, double phase, const PulseDev& p) {
    if constexpr (ENV == 0) {
        const double c = cos(M_PI * zeta / p.L);
        return sin(2.0 * M_PI * zeta / p.lambda - phase) * (c * c);
    }
    const double nl = p.ncycles * p.lambda;
    return sin(2.0 * M_PI * zeta / p.lambda - phase) * exp(-zeta * zeta * log(4.0) / (nl * nl));
}

// Sampled spectrum: S(zeta) = sum_m a_m exp(i (phi_m - w_m zeta)), evaluated
// as exp(-i w0 zeta) P(exp(-i dw zeta)) with P(z) = sum_m c_m z^m by Horner's
// rule (|z| = 1, so the rounding stays at a few ulps of sum |c_m|).  The
// profile of a part with carrier phase ph is Re[exp(i (ph + pi/2)) S] / gnorm.
__device__ void spectral_sum(double zeta, const PulseDev& p, double& sr, double& si) {
    const double* c = p.spec + 2;
    const int K = p.nfreq;
    double zs, zc, es, ec;
    sincos(-p.spec[1] * zeta, &zs, &zc);
    sincos(-p.spec[0] * zeta, &es, &ec);
    double pr = c[2 * (K - 1)], pim = c[2 * (K - 1) + 1];
    for (int m = K - 2; m >= 0; --m) {
        const double tr = pr * zc - pim * zs;
        const double ti = pr * zs + pim * zc;
        pr = c[2 * m] + tr;
        pim = c[2 * m + 1] + ti;
    }
    sr = pr * ec - pim * es;
    si = pr * es + pim * ec;
}

// The same sum from the interval polynomials: zeta in [-L/2, L/2] falls in
// interval q at t in [-1, 1) half widths from its centre, and S is the
// degree-7 Taylor polynomial in t with the interval's 8 complex
// coefficients: one 128-byte line and 14 fused multiply-adds per node in
// place of Horner's rule over all (about 200) samples.
__device__ __forceinline__ void spectral_poly(double zeta, const PulseDev& p, double& sr, double& si) {
    const double s = (zeta + 0.5 * p.L) * p.poly_inv;
    int q = (int)s;
    q = q < 0 ? 0 : (q >= p.npoly ? p.npoly - 1 : q);
    const double t = 2.0 * (s - q) - 1.0;
    const double2* c = reinterpret_cast<const double2*>(p.poly) + q * SPEC_COEF;
    double2 r = c[SPEC_COEF - 1];
#pragma unroll
    for (int k = SPEC_COEF - 2; k >= 0; --k) {
        const double2 ck = c[k];
        r.x = fma(r.x, t, ck.x);
        r.y = fma(r.y, t, ck.y);
    }
    sr = r.x;
    si = r.y;
}

// Coefficients of one interval per wave: lane m takes the samples m, m + 64,
// ... and adds c_m exp(-i w_m zc) (-i w_m h)^k / k! (h the half width, zc
// the centre), then the lanes are summed.  The phase w_m zc is the exact
// product (its rounding error is put back to first order).
__global__ __launch_bounds__(64) void k_spec_poly(double* __restrict__ poly, PulseDev p) {
    const int q = blockIdx.x, lane = threadIdx.x;
    const double h = 0.5 * p.L / p.npoly;
    const double zc = fma((double)(2 * q + 1), h, -0.5 * p.L);
    double a[2 * SPEC_COEF];
#pragma unroll
    for (int k = 0; k < 2 * SPEC_COEF; ++k) a[k] = 0.0;
    for (int m = lane; m < p.nfreq; m += 64) {
        const double w = fma((double)m, p.spec[1], p.spec[0]);
        const double ph = w * zc, err = fma(w, zc, -ph);
        double sn, cs;
        sincos(ph, &sn, &cs);
        const double ec = fma(-err, sn, cs), es = -fma(err, cs, sn);     // exp(-i w zc)
        const double cr = p.spec[2 + 2 * m], ci = p.spec[3 + 2 * m];
        double vr = fma(cr, ec, -(ci * es)), vi = fma(cr, es, ci * ec);
        const double wh = w * h;
#pragma unroll
        for (int k = 0; k < SPEC_COEF; ++k) {
            a[2 * k] += vr;
            a[2 * k + 1] += vi;
            const double f = wh / (k + 1), t = vr;                        // times -i wh / (k + 1)
            vr = vi * f;
            vi = -t * f;
        }
    }
#pragma unroll
    for (int k = 0; k < 2 * SPEC_COEF; ++k)
        for (int off = 32; off > 0; off >>= 1) a[k] += __shfl_xor(a[k], off);
    if (lane == 0) {
#pragma unroll
        for (int k = 0; k < 2 * SPEC_COEF; ++k) poly[(long)q * 2 * SPEC_COEF + k] = a[k];
    }
}

// Wavefront phase of the direction (alpha, azimuth): a sum of Gaussian bumps
// over the angular position (ay, az) = alpha (y, z) / rho (Sec. III.B.3).
__device__ double bump_phase(double alpha, double y, double z, double rho, const PulseDev& p) {
    const double ay = rho > 0.0 ? alpha * y / rho : 0.0;
    const double az = rho > 0.0 ? alpha * z / rho : 0.0;
    double ph = 0.0;
    for (int i = 0; i < p.nbumps; ++i) {
        const double* bp = p.bumps + 4 * i;
        const double dy = ay - bp[0], dz = az - bp[1];
        ph += bp[2] * exp(-(dy * dy + dz * dz) / (bp[3] * bp[3]));
    }
    return ph;
}

// Adds the unmapped pulse at physical point (x, y, z), rho = sqrt(y^2 + z^2),
// to e, b.  Points clearly outside the aperture, and points clearly inside
// the flat part of a flat-top aperture, are told by -x against rho
// cot(angle) (1e-9 R to the safe side); the angle itself is evaluated only
// for the others and where the profile needs it.  ENV and BUMPS are template
// parameters because the float64 trigonometry of the profiles not in use
// would otherwise take registers in every variant.
enum EnvKind { ENV_COS2 = 0, ENV_GAUSS = 1, ENV_SUM = 2, ENV_POLY = 3 };
template <int ENV, bool BUMPS>
__device__ __forceinline__ void add_pulse(double x, double y, double z, double rho, const PulseDev& p, double* e, double* b) {
    const double R = sqrt(x * x + y * y + z * z);
    const double zeta = R - p.R0;
    if (!(zeta >= -0.5 * p.L && zeta <= 0.5 * p.L)) return;
    const double tol = 1e-9 * R;
    if (-x < rho * p.cot_max - tol) return;
    double ts = 1.0, alpha = 0.0;
    if (BUMPS || !(-x > rho * p.cot_lo + tol)) {
        alpha = atan2(rho, -x);                             // angle from the -x axis
        if (!(alpha <= p.alpha_max)) return;
        ts = u_ts(alpha, p);
    }
    double sr = 0.0, si = 0.0;                              // shared by both polarisation parts
    if constexpr (ENV == ENV_POLY) spectral_poly(zeta, p, sr, si);
    if constexpr (ENV == ENV_SUM) spectral_sum(zeta, p, sr, si);
    // the perturbation adds to every part's carrier phase, as the CEP does
    double dph = 0.0, cb = 1.0, sb = 0.0;
    if constexpr (BUMPS) {
        dph = bump_phase(alpha, y, z, rho, p);
        if constexpr (ENV >= ENV_SUM) sincos(dph, &sb, &cb);
    }
    const double iR = 1.0 / R;
    for (int k = 0; k < p.nparts; ++k) {
        double ul;
        if constexpr (ENV >= ENV_SUM)
            ul = ((p.cph[k] * cb - p.sph[k] * sb) * sr - (p.sph[k] * cb + p.cph[k] * sb) * si) / p.gnorm;
        else
            ul = u_l_closed<ENV>(zeta, p.cep + p.phase_off[k] + dph, p);
        const double u = p.A * iR * ul * ts;
        const double* d = p.d[k];
        // s1 ~ d x R, s0 ~ R x (d x R)
        const double c1x = d[1] * z - d[2] * y, c1y = d[2] * x - d[0] * z, c1z = d[0] * y - d[1] * x;
        const double n1 = sqrt(c1x * c1x + c1y * c1y + c1z * c1z);
        if (!(n1 > 0.0)) continue;
        const double c0x = y * c1z - z * c1y, c0y = z * c1x - x * c1z, c0z = x * c1y - y * c1x;
        const double au = p.amp[k] * u;
        const double i1 = 1.0 / n1, i0 = i1 * iR;
        e[0] += au * c0x * i0; e[1] += au * c0y * i0; e[2] += au * c0z * i0;
        b[0] += au * c1x * i1; b[1] += au * c1y * i1; b[2] += au * c1z * i1;
    }
}

// Layer nodes: sum of the pulse over the preimages x + n D, n ascending
// (Eq. (13) inverted; overlapping replicas superpose); with transverse
// replication also over y + m Dy, z + l Dz (l, then m ascending outside the
// x preimages).  A thread takes V consecutive nodes of a row (16 bytes of
// each component; every supported nx is a multiple of 8), so the row's
// geometry is evaluated once for them.  At a given rho the support is an
// interval of x, [-sqrt(R_max^2 - rho^2), -max(rho cot(alpha_max), x_rc)], so
// only the one or two n that reach it are tried (1e-9 R_max to the safe
// side; add_pulse decides).  Bound by float64 arithmetic (geometry and the
// interval polynomial) in float32, by the stores in float64.  MI355X, before
// (a node per thread, every preimage tried, the sum over all samples) and
// now: spectral 96 x 256 x 256 float32 765 -> 88 us, 512^3 4870 -> 826 us;
// cos^2 128 x 1024^2 float32 2142 -> 735 us, 112 x 896^2 float64 1652 -> 690
// us (6.2 TB/s).  One or two nodes per thread: 512^3 1.7 and 1.4 times this
// layout's time.  Four blocks per CU (128 registers) for the polynomial
// (887 -> 826 us); the others would spill.
template <typename T, int ENV, bool BUMPS>
__global__ __launch_bounds__(256, ENV == ENV_POLY && !BUMPS ? 4 : 1) void k_init_map(T* __restrict__ state, GridDev g, PulseDev p) {
    constexpr int V = 16 / sizeof(T);
    typedef T vec __attribute__((ext_vector_type(V)));
    const unsigned vx = (unsigned)g.nx / V;
    const unsigned id = blockIdx.x * 256u + threadIdx.x;       // at most 2^30 nodes (1024 per axis)
    const unsigned row = id / vx;
    if (row >= (unsigned)g.ny * (unsigned)g.nz) return;
    const int i = (int)(id - row * vx) * V;
    const int k = (int)(row / (unsigned)g.ny);
    const int j = (int)(row - (unsigned)k * (unsigned)g.ny);
    const double D = g.nx * g.dx;
    const double y = g.y_min + j * g.dy;
    const double z = g.z_min + k * g.dz;
    const double Rmax = p.R0 + 0.5 * p.L, slack = 1e-9 * Rmax, iD = 1.0 / D;
    const double Dy = g.ny * g.dy, Dz = g.nz * g.dz;
    long m0 = 0, m1 = 0, l0 = 0, l1 = 0;
    if (g.rep_yz) {
        m0 = (long)floor((-Rmax - y) / Dy) - 1;
        m1 = (long)ceil((Rmax - y) / Dy) + 1;
        l0 = (long)floor((-Rmax - z) / Dz) - 1;
        l1 = (long)ceil((Rmax - z) / Dz) + 1;
    }
    // the x range of the support at a transverse point; empty (lo > hi) outside R_max
    auto support = [&](double yy, double zz, double& rho, double& lo, double& hi) {
        const double rho2 = yy * yy + zz * zz;
        lo = 1.0; hi = -1.0; rho = 0.0;
        if (rho2 <= Rmax * Rmax) {
            rho = sqrt(rho2);
            const double xm = sqrt(Rmax * Rmax - rho2);
            lo = -xm - slack;
            hi = fmin(xm, -fmax(rho * p.cot_max, p.x_rc)) + slack;
        }
    };
    double rho, lo, hi;
    if (!g.rep_yz) support(y, z, rho, lo, hi);
    vec o[6];
#pragma unroll
    for (int c = 0; c < 6; ++c)
#pragma unroll
        for (int v = 0; v < V; ++v) o[c][v] = T(0);
#pragma unroll 1
    for (int v = 0; v < V; ++v) {
        const double xt = g.x_min + (i + v) * g.dx;
        double e[3] = {0.0, 0.0, 0.0}, b[3] = {0.0, 0.0, 0.0};
        for (long l = l0; l <= l1; ++l)
            for (long m = m0; m <= m1; ++m) {
                const double yy = g.rep_yz ? y + m * Dy : y, zz = g.rep_yz ? z + l * Dz : z;
                if (g.rep_yz) support(yy, zz, rho, lo, hi);
                if (lo <= hi) {
                    const long n0 = (long)ceil((lo - xt) * iD), n1 = (long)floor((hi - xt) * iD);
                    for (long n = n0; n <= n1; ++n) add_pulse<ENV, BUMPS>(xt + n * D, yy, zz, rho, p, e, b);
                }
            }
        // one copy of the pulse's code for all V nodes: the node's results
        // are selected into its place
#pragma unroll
        for (int c = 0; c < 6; ++c)
#pragma unroll
            for (int w = 0; w < V; ++w) o[c][w] = w == v ? T(c < 3 ? e[c] : b[c - 3]) : o[c][w];
    }
    const size_t cells = (size_t)g.nx * g.ny * g.nz;
    T* dst = state + (size_t)row * g.nx + i;
#pragma unroll
    for (int c = 0; c < 6; ++c) *reinterpret_cast<vec*>(dst + c * cells) = o[c];
}

// ---------------------------------------------------------------- cut-out
// Coordinate of node I along an axis.  When the origin is a node (lo / d an
// integer), the coordinate is the node's integer offset from the origin
// times d, so grids that share the spacing give the very same value to the
// same point, and the cut-out of Eq. (15) decides nodes on its spheres
// (R = L, R = r(t), ...) alike in every such grid.
__device__ double node_coord(long I, double lo, double d) {
    const double o = lo / d, r = rint(o);
    return fabs(o - r) <= 1e-6 ? (double)(I + (long)r) * d : lo + I * d;
}

// I_S(t)(R) of Eq. (15), third case read as "x >= 0 and R > r(t)".
__device__ bool cutout_keep(double x, double y, double z, double t, double Rmin, double Rmax) {
    const double R = sqrt(x * x + y * y + z * z);
    const double L = Rmax - Rmin;
    const double l = -Rmax + t, r = -Rmin + t;
    if (r < 0.0) return !((R >= -l) || (R < -r) || (x > 0.0));
    if (l <= 0.0) return !(((x < 0.0) && (R > L)) || ((x >= 0.0) && (R > r)));
    return !((R <= l) || (R > r) || (x < 0.0));
}

template <typename T>
__global__ __launch_bounds__(256) void k_readout(const T* __restrict__ state, T* __restrict__ out, GridDev g,
                                                 int wx, int wy, int wz, long ic, long jc, long kc,
                                                 double t, double Rmin, double Rmax) {
    const long wn = (long)wx * wy * wz;
    const long id = (long)blockIdx.x * blockDim.x + threadIdx.x;
    if (id >= wn) return;
    const int a = (int)(id % wx), bj = (int)((id / wx) % wy), ck = (int)(id / ((long)wx * wy));
    const long I = ic + a - wx / 2, J = jc + bj - wy / 2, K = kc + ck - wz / 2;
    long ix = I % g.nx;
    if (ix < 0) ix += g.nx;
    long jy = J, kz = K;
    if (g.rep_yz) {
        jy = J % g.ny;
        if (jy < 0) jy += g.ny;
        kz = K % g.nz;
        if (kz < 0) kz += g.nz;
    }
    const double x = node_coord(I, g.x_min, g.dx), y = node_coord(J, g.y_min, g.dy), z = node_coord(K, g.z_min, g.dz);
    const bool keep = cutout_keep(x, y, z, t, Rmin, Rmax);
    const long cells = (long)g.nx * g.ny * g.nz;
    const long src = (kz * g.ny + jy) * g.nx + ix;
    for (int c = 0; c < 6; ++c) out[c * wn + id] = keep ? state[c * cells + src] : T(0);
}

// ---------------------------------------------------------------- reductions
template <typename T>
__global__ __launch_bounds__(256) void k_sumsq(const T* __restrict__ x, size_t n, double* __restrict__ part) {
    __shared__ double red[4];
    double acc = 0.0;
    for (size_t i = (size_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (size_t)gridDim.x * 256) {
        const double v = double(x[i]);
        acc += v * v;
    }
    for (int off = 32; off > 0; off >>= 1) acc += __shfl_xor(acc, off);
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = acc;
    __syncthreads();
    if (threadIdx.x == 0) part[blockIdx.x] = ((red[0] + red[1]) + red[2]) + red[3];
}

__global__ __launch_bounds__(256) void k_reduce(const double* __restrict__ part, int m, int stride, int offset,
                                                int op, double* __restrict__ out) {
    __shared__ double red[4];
    double acc = 0.0;
    for (int i = threadIdx.x; i < m; i += 256) {
        const double v = part[(long)i * stride + offset];
        acc = op == 0 ? acc + v : fmax(acc, v);
    }
    for (int off = 32; off > 0; off >>= 1) {
        const double o = __shfl_xor(acc, off);
        acc = op == 0 ? acc + o : fmax(acc, o);
    }
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = acc;
    __syncthreads();
    if (threadIdx.x == 0) {
        *out = op == 0 ? ((red[0] + red[1]) + red[2]) + red[3]
                       : fmax(fmax(red[0], red[1]), fmax(red[2], red[3]));
    }
}

// ---------------------------------------------------------------- launchers
template <typename T>
hipError_t launch_init_map(T* state, const GridDev& g, const PulseDev& p, hipStream_t st) {
    const long items = (long)g.nx * g.ny * g.nz / (16 / sizeof(T));
    const unsigned nb = (unsigned)((items + 255) / 256);
    const int env = p.envelope == 0 ? ENV_COS2 : p.envelope == 1 ? ENV_GAUSS : p.npoly > 0 ? ENV_POLY : ENV_SUM;
#define TF_INIT(E)                                                                                          \
    case E:                                                                                                 \
        if (p.nbumps > 0) hipLaunchKernelGGL((k_init_map<T, E, true>), dim3(nb), dim3(256), 0, st, state, g, p); \
        else hipLaunchKernelGGL((k_init_map<T, E, false>), dim3(nb), dim3(256), 0, st, state, g, p);        \
        break;
    switch (env) {
        TF_INIT(ENV_COS2)
        TF_INIT(ENV_GAUSS)
        TF_INIT(ENV_SUM)
        TF_INIT(ENV_POLY)
    }
#undef TF_INIT
    return hipGetLastError();
}

hipError_t launch_spec_poly(double* poly, const PulseDev& p, hipStream_t st) {
    hipLaunchKernelGGL(k_spec_poly, dim3(p.npoly), dim3(64), 0, st, poly, p);
    return hipGetLastError();
}

template <typename T>
hipError_t launch_readout(const T* state, T* out, const GridDev& g, int wx, int wy, int wz, long ic, long jc,
                          long kc, double t, double R_min, double R_max, hipStream_t st) {
    const long wn = (long)wx * wy * wz;
    const unsigned nb = (unsigned)((wn + 255) / 256);
    hipLaunchKernelGGL(k_readout<T>, dim3(nb), dim3(256), 0, st, state, out, g, wx, wy, wz, ic, jc, kc, t,
                       R_min, R_max);
    return hipGetLastError();
}

template <typename T>
hipError_t launch_sumsq(const T* x, size_t n, double* partials, int nb, hipStream_t st) {
    hipLaunchKernelGGL(k_sumsq<T>, dim3(nb), dim3(256), 0, st, x, n, partials);
    return hipGetLastError();
}

hipError_t launch_reduce(const double* partials, int m, int stride, int offset, int op, double* out,
                         hipStream_t st) {
    hipLaunchKernelGGL(k_reduce, dim3(1), dim3(256), 0, st, partials, m, stride, offset, op, out);
    return hipGetLastError();
}

template hipError_t launch_init_map<float>(float*, const GridDev&, const PulseDev&, hipStream_t);
template hipError_t launch_init_map<double>(double*, const GridDev&, const PulseDev&, hipStream_t);
template hipError_t launch_readout<float>(const float*, float*, const GridDev&, int, int, int, long, long, long,
                                          double, double, double, hipStream_t);
template hipError_t launch_readout<double>(const double*, double*, const GridDev&, int, int, int, long, long,
                                           long, double, double, double, hipStream_t);
template hipError_t launch_sumsq<float>(const float*, size_t, double*, int, hipStream_t);
template hipError_t launch_sumsq<double>(const double*, size_t, double*, int, hipStream_t);

}  // namespace tf
