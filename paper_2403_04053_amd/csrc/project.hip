// Near-to-distant-field projection over the virtual box (Section 3.2).
//
// All sums are FP64.  Both outputs are linear in the phasors of each face
// plane, through the trigonometric interpolant of Eq. AnBottomPsi; its DFT is
// folded into the tables below, so no plane is transformed on a call.
//
//  * far field: the cell formula of Eqs. bottomPsi_lm ... leftrightPsi_ln in
//    the limit of Eq. FDTDfarfieldapprox.  For a direction r_hat every cell
//    term factors into an in-plane b-part and c-part, so a face contributes
//    h_c(r_c)^T [P_dpsi + i r_a P_psi] h_b(r_b).  Each factor is an entire
//    function of its component of exponential type X, the box's reduced half
//    width, so its Chebyshev series on [-1, 1] ends, to rounding, a little
//    past X: a face is a K x K matrix of coefficients (two small GEMMs per
//    plane and call) and a direction costs sum_jk C_jk T_j(r_c) T_k(r_b), real
//    times complex, on the FP64 matrix cores;
//  * Fresnel points: each sinc of the cell formula is expanded to 8th order
//    in its shift alpha = k d R_hat / 2, so the spectral double sum of a cell
//    becomes sum_pq alpha_b^p alpha_c^q Q_pq(cell); the Q tables are two
//    batched GEMMs per face and field.  The 36 terms of total degree 9 to 16
//    are economised onto the 45 of degree 8 and less, and the per-point work
//    is a Horner evaluation per cell with the exact distance R and
//    exp(ikR)/R.
//
// Reduced units throughout (k = 1); the far-field amplitude is divided by k0
// at the end to return physical length units.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <string>
#include <vector>

#include "fp64_math.hpp"
#include "internal.hpp"
#include "project.hpp"

namespace pstd {

namespace {

constexpr double kPi = 3.141592653589793238462643383279502884;
constexpr int kOrder = 8;            // sinc expansion order
constexpr int kTerms = kOrder + 1;
constexpr int kPairs = kTerms * kTerms;               // (p, q), p, q <= 8
constexpr int kLow = kTerms * (kTerms + 1) / 2;       // those with p + q <= 8
constexpr int kHigh = kPairs - kLow;
// row p of the low terms starts here: (p, 0), (p, 1), ... (p, 8 - p)
__host__ __device__ constexpr int low_row(int p) { return p * kTerms - p * (p - 1) / 2; }

__host__ __device__ inline int face_axis_b(int a) { return a == 0 ? 1 : 0; }
__host__ __device__ inline int face_axis_c(int a) { return a == 2 ? 1 : 2; }

__device__ __forceinline__ double2 zmul(double2 a, double2 b) {
    return make_double2(a.x * b.x - a.y * b.y, a.x * b.y + a.y * b.x);
}
__device__ __forceinline__ double2 zadd(double2 a, double2 b) { return make_double2(a.x + b.x, a.y + b.y); }

// ---------------------------------------------------------------------------
// phasor finalisation: the six faces in one launch
// ---------------------------------------------------------------------------

struct FinalizeArgs {
    const double2* acc[3];
    int64_t points[3];
    int blocks[3];  // of one face
};

__global__ void finalize_kernel(FinalizeArgs f, double2 sv, double2 sd, double2* __restrict__ out) {
    int b = (int)blockIdx.x, a = 0;
    while (a < 2 && b >= 2 * f.blocks[a]) {
        b -= 2 * f.blocks[a];
        out += 4 * f.points[a];
        ++a;
    }
    const int side = b >= f.blocks[a];
    const int64_t points = f.points[a];
    const int64_t i = (int64_t)(b - side * f.blocks[a]) * blockDim.x + threadIdx.x;
    if (i >= points) return;
    out += 2 * side * points;
    const double2* base = f.acc[a] + (int64_t)side * 4 * points;
    const double2 s0 = base[i], c0 = base[points + i], s1 = base[2 * points + i], c1 = base[3 * points + i];
    const double ar = s0.x + c0.x, ai = s0.y + c0.y, br = s1.x + c1.x, bi = s1.y + c1.y;
    out[i] = make_double2(ar * sv.x - ai * sv.y, ar * sv.y + ai * sv.x);
    out[points + i] = make_double2(br * sd.x - bi * sd.y, br * sd.y + bi * sd.x);
}

// W[m][i] = exp(-2 pi i m i / N), the plane DFT as a matrix
__global__ void dft_matrix_kernel(int N, double2* __restrict__ W) {
    const int64_t id = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (id >= (int64_t)N * N) return;
    const int64_t j = ((id / N) * (id % N)) % N;
    double sn, cs;
    sincospi(2.0 * (double)j / N, &sn, &cs);
    W[id] = make_double2(cs, -sn);
}

// ---------------------------------------------------------------------------
// batched complex GEMM on the FP64 matrix cores, row-major:
// C[i][j] = sum_k A[i][k] B[k][j]; TA: A is given as [k][i], TB: B as [j][k];
// CA, CB: the conjugate of A, B
//
// v_mfma_f64_16x16x4f64 takes, per lane l, A[i][k] with i = l % 16, k = l / 16
// and B[k][j] with j = l % 16, k = l / 16, and leaves D[i][j] in register r
// of lane l for i = 4 r + l / 16, j = l % 16.  A complex product is four real
// ones: re += Ar Br - Ai Bi, im += Ar Bi + Ai Br.  A workgroup (4 waves)
// computes a T x T tile, each wave a quarter of it (U x U MFMA tiles), from
// 16-deep slices of A and B staged in LDS, the next slice's loads in flight
// during the products.  The matrices here are a few tiles each, so the batch
// (two levels of strides) is what fills the chip: one launch takes every
// (field, p, q) of a face, and where that gives 64 x 64 tiles to fewer than
// half of the CUs, tiles of 32 x 32 (a quarter of the work per slice) shorten
// the chain of slices: 160 x 92 x 160, batch 4: 25.3 us with 64, 11.2 us with 32.
// ---------------------------------------------------------------------------

typedef double v4d __attribute__((ext_vector_type(4)));

constexpr int ZK = 16;   // K slice

// one operand of a batched product: leading dimension and the strides of the
// inner and outer batch index
struct ZOp {
    const double2* p;
    int64_t ld, s0 = 0, s1 = 0;
};

template <int T, bool TA, bool CA, bool TB, bool CB>
__global__ __launch_bounds__(256) void zgemm_kernel(int M, int N, int K, ZOp a_, ZOp b_, ZOp c_, int n0) {
    constexpr int U = T / 32;            // MFMA tiles per wave and axis
    constexpr int LD = T * ZK / 256;     // elements per thread, slice and operand
    __shared__ double2 As[T][ZK + 1];
    __shared__ double2 Bs[ZK][T + 1];
    const int z0 = (int)blockIdx.z % n0, z1 = (int)blockIdx.z / n0;
    const double2* __restrict__ A = a_.p + z0 * a_.s0 + z1 * a_.s1;
    const double2* __restrict__ B = b_.p + z0 * b_.s0 + z1 * b_.s1;
    double2* __restrict__ C = const_cast<double2*>(c_.p) + z0 * c_.s0 + z1 * c_.s1;
    const int64_t lda = a_.ld, ldb = b_.ld, ldc = c_.ld;
    const int i0 = blockIdx.y * T, j0 = blockIdx.x * T;
    const int t = threadIdx.x;
    const int lane = t & 63, wave = t >> 6;
    const int wi = (wave >> 1) * (T / 2), wj = (wave & 1) * (T / 2);
    const int li = lane & 15, lk = lane >> 4;
    v4d re[U][U], im[U][U];
#pragma unroll
    for (int u = 0; u < U; ++u)
#pragma unroll
        for (int v = 0; v < U; ++v) {
            re[u][v] = v4d{0, 0, 0, 0};
            im[u][v] = v4d{0, 0, 0, 0};
        }
    double2 ra[LD], rb[LD];
    auto load = [&](int k0) {
#pragma unroll
        for (int n = 0; n < LD; ++n) {
            const int e = t + n * 256;
            {
                const int r = TA ? e % T : e / ZK, c = TA ? e / T : e % ZK;
                const int gi = i0 + r, gk = k0 + c;
                double2 x = make_double2(0, 0);
                if (gi < M && gk < K) x = A[TA ? (int64_t)gk * lda + gi : (int64_t)gi * lda + gk];
                if (CA) x.y = -x.y;
                ra[n] = x;
            }
            {
                const int r = TB ? e % ZK : e / T, c = TB ? e / ZK : e % T;
                const int gk = k0 + r, gj = j0 + c;
                double2 x = make_double2(0, 0);
                if (gk < K && gj < N) x = B[TB ? (int64_t)gj * ldb + gk : (int64_t)gk * ldb + gj];
                if (CB) x.y = -x.y;
                rb[n] = x;
            }
        }
    };
    load(0);
    for (int k0 = 0; k0 < K; k0 += ZK) {
#pragma unroll
        for (int n = 0; n < LD; ++n) {
            const int e = t + n * 256;
            As[TA ? e % T : e / ZK][TA ? e / T : e % ZK] = ra[n];
            Bs[TB ? e % ZK : e / T][TB ? e / ZK : e % T] = rb[n];
        }
        __syncthreads();
        if (k0 + ZK < K) load(k0 + ZK);
#pragma unroll
        for (int ks = 0; ks < ZK; ks += 4) {
            double2 a[U], b[U];
#pragma unroll
            for (int u = 0; u < U; ++u) a[u] = As[wi + u * 16 + li][ks + lk];
#pragma unroll
            for (int v = 0; v < U; ++v) b[v] = Bs[ks + lk][wj + v * 16 + li];
#pragma unroll
            for (int u = 0; u < U; ++u)
#pragma unroll
                for (int v = 0; v < U; ++v) {
                    re[u][v] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[u].x, b[v].x, re[u][v], 0, 0, 0);
                    re[u][v] = __builtin_amdgcn_mfma_f64_16x16x4f64(-a[u].y, b[v].y, re[u][v], 0, 0, 0);
                    im[u][v] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[u].x, b[v].y, im[u][v], 0, 0, 0);
                    im[u][v] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[u].y, b[v].x, im[u][v], 0, 0, 0);
                }
        }
        __syncthreads();
    }
#pragma unroll
    for (int u = 0; u < U; ++u)
#pragma unroll
        for (int v = 0; v < U; ++v)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int gi = i0 + wi + u * 16 + 4 * r + lk, gj = j0 + wj + v * 16 + li;
                if (gi < M && gj < N) C[(int64_t)gi * ldc + gj] = make_double2(re[u][v][r], im[u][v][r]);
            }
}

struct ZOpts {
    bool ta = false, ca = false, tb = false, cb = false;
};

template <int T>
hipError_t zgemm_tile(int M, int N, int K, ZOp A, ZOp B, ZOp C, int n0, int n1, ZOpts o, hipStream_t stream) {
    const dim3 grid((N + T - 1) / T, (M + T - 1) / T, n0 * n1);
    auto go = [&](auto kernel) { hipLaunchKernelGGL(kernel, grid, dim3(256), 0, stream, M, N, K, A, B, C, n0); };
    // the forms in use
    if (o.ta && o.ca && !o.tb && !o.cb) go(zgemm_kernel<T, true, true, false, false>);
    else if (!o.ta && !o.ca && o.tb && !o.cb) go(zgemm_kernel<T, false, false, true, false>);
    else if (!o.ta && !o.ca && !o.tb && o.cb) go(zgemm_kernel<T, false, false, false, true>);
    else if (!o.ta && !o.ca && !o.tb && !o.cb) go(zgemm_kernel<T, false, false, false, false>);
    else return hipErrorInvalidValue;
    return hipGetLastError();
}

hipError_t zgemm(int M, int N, int K, ZOp A, ZOp B, double2* Cp, int64_t ldc, int64_t sc0, int64_t sc1, int n0, int n1,
                 ZOpts o, hipStream_t stream) {
    if (M <= 0 || N <= 0 || n0 <= 0 || n1 <= 0) return hipSuccess;
    const ZOp C{Cp, ldc, sc0, sc1};
    const int64_t groups = (int64_t)((N + 63) / 64) * ((M + 63) / 64) * n0 * n1;
    return groups < 128 ? zgemm_tile<32>(M, N, K, A, B, C, n0, n1, o, stream)
                        : zgemm_tile<64>(M, N, K, A, B, C, n0, n1, o, stream);
}

// ---------------------------------------------------------------------------
// far field
// ---------------------------------------------------------------------------

// One axis of the box as the far field sees it: N points of spacing d, the
// face's cells between grid indices lo and hi
struct FarAxis {
    int N, lo, hi;
    double d;
    double mid, half;  // centre and half width of the cells
};

// the product x y as a rounded value and its rounding error
__device__ __forceinline__ double two_product(double x, double y, double* err) {
    const double p = x * y;
    *err = fma(x, y, -p);
    return p;
}

// sine and cosine of p + e, e within a few of p's last digits
__device__ __forceinline__ void sincos_sum(double p, double e, double* sn, double* cs) {
    double s, c;
    sincos(p, &s, &c);
    *sn = fma(e, c, s);
    *cs = fma(-e, s, c);
}

// g(m) = (-1)^b' sinc(theta) sum_{l=lo}^{hi-1} exp(2 i theta (x_l / d)), theta =
// pi b'/N - d r/2, b' the signed index of m, x_l = (l - N/2 + 1/2) d.  With the
// closed form of the geometric sum that is (-1)^b' sin(M theta) / theta times the
// phase of the middle, M = hi - lo.  centred: without the factor exp(-i r mid).
// theta is carried with its rounding error, as are the nodes r + r_low, the faces'
// phases and the directions' angles: a rounded product of 50 radians is off by
// 3.5e-15, a rounded node moves it by 2e-15.  RMS error of far fields of random planes
// against 80-bit sums, of their RMS (with rounded nodes; with the factors themselves
// and rounded products, direction by direction): 160^3 2.0e-15 (3.4, 3.9), 64 x 96 x 108
// 1.5e-15 (2.6, 2.5), 288 x 48 x 64 at 3 points per wavelength 6.4e-15 (14.9, 15.1).
__device__ __forceinline__ double2 far_factor(const FarAxis& ax, double r, double r_low, int m, bool centred) {
    const int bp = m < ax.N / 2 ? m : m - ax.N;
    const int M = ax.hi - ax.lo;
    constexpr double kPiLow = 1.2246467991473532e-16;  // pi - kPi
    double e1, e2;
    const double p1 = two_product(kPi, bp, &e1);
    const double t1 = p1 / ax.N;
    const double l1 = (fma(-t1, ax.N, p1) + fma(kPiLow, bp, e1)) / ax.N;
    const double t2 = two_product(r, 0.5 * ax.d, &e2);
    const double th = t1 - t2, v = th - t1;
    const double tl = ((t1 - (th - v)) - (t2 + v)) + (l1 - fma(r_low, 0.5 * ax.d, e2));
    double em;
    const double pm = two_product(M, th, &em);
    double sm, cm;
    sincos_sum(pm, fma(M, tl, em), &sm, &cm);
    const double theta = th + tl;
    const double mag = (theta == 0.0 ? (double)M : sm / theta) * ((bp & 1) ? -1.0 : 1.0);
    // 2 pi b' mid / (N d), the angle reduced in integers
    const int64_t q = (int64_t)bp * (ax.lo + ax.hi - ax.N) % (2 * (int64_t)ax.N);
    double sn, cs;
    sincospi((double)q / ax.N, &sn, &cs);
    if (!centred) {
        double er, sr, cr;
        const double pr = two_product(-r, ax.mid, &er);
        sincos_sum(pr, er, &sr, &cr);
        const double2 f = zmul(make_double2(cs, sn), make_double2(cr, sr));
        cs = f.x;
        sn = f.y;
    }
    return make_double2(mag * cs, mag * sn);
}

// G[j][m]: the centred factor at the Chebyshev nodes r_j = cos(pi (j + 1/2) / K),
// node[j] as a rounded value and the rest of it (80-bit values of the host)
__global__ void far_nodes_kernel(FarAxis ax, int K, const double2* __restrict__ node, double2* __restrict__ G) {
    const int64_t id = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (id >= (int64_t)K * ax.N) return;
    const int m = (int)(id % ax.N), j = (int)(id / ax.N);
    G[id] = far_factor(ax, node[j].x, node[j].y, m, true);
}

// D[k][j]: values at the K nodes to Chebyshev coefficients
__global__ void far_dct_kernel(int K, double2* __restrict__ D) {
    const int64_t id = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (id >= (int64_t)K * K) return;
    const int64_t k = id / K, j = id % K;
    // cos(k pi (j + 1/2) / K), the angle reduced in integers
    const int64_t q = (k * (2 * j + 1)) % (4 * K);
    D[id] = make_double2((k ? 2.0 : 1.0) / K * cospi((double)q / (2 * K)), 0.0);
}

// coefficients of one axis's two faces in the order the direction kernel
// reads: [k (Kb, padded to 4)][j (Kc, padded to 16)][side][psi, dpsi][re, im],
// zero in the padding; C: [side][psi, dpsi][Kc][Kb]
__global__ void far_pack_kernel(int Kb, int Kc, int Kbp, int Kcp, const double2* __restrict__ C,
                                double2* __restrict__ out) {
    const int64_t id = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (id >= (int64_t)Kbp * Kcp * 4) return;
    const int sf = (int)(id & 3);
    const int j = (int)((id >> 2) % Kcp), k = (int)((id >> 2) / Kcp);
    out[id] = j < Kc && k < Kb ? C[((int64_t)sf * Kc + j) * Kb + k] : make_double2(0, 0);
}

struct FarEval {
    const double* coef;  // far_pack_kernel's output of this axis
    int Kbp, Kcp;
    double half, half_err;  // of the normal axis: the faces lie at mid -+ (half + half_err)
    double pref;
};
struct FarArgs {
    FarEval ax[3];
    int jsplit;
};

// sum_jk C_jk T_j(r_c) T_k(r_b) of one axis's two faces for 16 directions per
// wave: the sum over k is a product of [16 directions x Kb] by [Kb x 16 j] for
// each of the eight numbers (side, field, re/im) on the FP64 matrix cores,
// T_k advancing by four k per step as a rotation in the lane that feeds it; the
// sum over j is taken from the accumulators with the faces' phases.  grid.y = axis
// * jsplit + part: few directions split the j tiles; row y of part receives the
// sums.  Bound by the matrix cores (three axes of about 92 x 96 coefficients: 65160
// directions in 545 us, 0.35 ms of it at their full rate; 3 waves per SIMD although
// 11 registers spill, 790 us at 2; 32 directions per wave, half the coefficient
// loads, at 2 waves without spills 583 against 587 us per call) and by what a wave
// computes first: with a direction's angle, rotation and phase in one lane instead
// of sixteen a call takes 571 instead of 587 us, 64^3 planes 260 instead of 278.  The
// former path, a complex product per 8192 directions and face with the factors
// themselves, took 7.3 ms in all.
constexpr int kFarWaves = 4;

// cos(k (pi/2 - a)) = T_k(sin a) and its companion -sin(k (pi/2 - a)) in *sn,
// which a rotation by 4 a (16 a) advances by four (sixteen) k: the quarter
// turns of k are exact
__device__ __forceinline__ void cheb_start(int k, double a, double* sn, double* cs) {
    double err, s, c;
    const double p = two_product(k, a, &err);
    sincos_sum(p, err, &s, &c);
    const int q = k & 3;
    *cs = q == 0 ? c : q == 1 ? s : q == 2 ? -c : -s;
    *sn = q == 0 ? s : q == 1 ? -c : q == 2 ? -s : c;
}


__global__ __launch_bounds__(64 * kFarWaves, 3) void far_eval_kernel(const double3* __restrict__ dirs, int64_t nd,
                                                                  FarArgs f, double2* __restrict__ part) {
    const int lane = threadIdx.x & 63, li = lane & 15, lk = lane >> 4;
    const int64_t d0 = ((int64_t)blockIdx.x * kFarWaves + (threadIdx.x >> 6)) * 16;
    if (d0 >= nd) return;  // whole wave
    const int a = (int)blockIdx.y / f.jsplit, js = (int)blockIdx.y % f.jsplit;
    const int b = face_axis_b(a), c = face_axis_c(a);
    const FarEval ev = f.ax[a];
    auto comp = [](double3 v, int i) { return i == 0 ? v.x : i == 1 ? v.y : v.z; };
    // r = cos(pi/2 - a): a, unlike the angle itself, keeps its relative precision
    // (directions beyond the interval are replaced afterwards)
    auto angle = [](double r) { return asin(fmin(1.0, fmax(-1.0, r))); };
    // feeder: direction li, k = lk + 4 step
    const double tb = angle(comp(dirs[min(d0 + li, nd - 1)], b));
    double c0, s0, c4, s4;
    cheb_start(lk, tb, &s0, &c0);
    sincos(4.0 * tb, &s4, &c4);
    // receiver: directions 4 r + lk, column j = 16 tile + li
    const int tiles = ev.Kcp / 16, per = (tiles + f.jsplit - 1) / f.jsplit;
    const int t0 = js * per, t1 = min(tiles, t0 + per);
    double tc[4], ts[4], c16[4], s16[4], ra[4], orr[4], oi[4];
    double2 w[4];
    {
        // a direction's angle, rotation and phase in one lane of each row of 16,
        // handed to the lanes that receive it
        const double3 v = dirs[min(d0 + li, nd - 1)];
        const double t = angle(comp(v, c)), rn = comp(v, a);
        double sn, cs, sr, cr, err;
        sincos(16.0 * t, &sr, &cr);
        const double ph = two_product(rn, ev.half, &err);
        sincos_sum(ph, fma(rn, ev.half_err, err), &sn, &cs);
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int from = 4 * r + lk;
            cheb_start(16 * t0 + li, __shfl(t, from, 64), &ts[r], &tc[r]);
            c16[r] = __shfl(cr, from, 64);
            s16[r] = __shfl(sr, from, 64);
            ra[r] = __shfl(rn, from, 64);
            // pref exp(i ra half) of the low face; the high face's is -conj of it
            w[r] = make_double2(ev.pref * __shfl(cs, from, 64), ev.pref * __shfl(sn, from, 64));
            orr[r] = 0;
            oi[r] = 0;
        }
    }
    for (int tile = t0; tile < t1; ++tile) {
        v4d acc[8];
#pragma unroll
        for (int q = 0; q < 8; ++q) acc[q] = v4d{0, 0, 0, 0};
        const double2* __restrict__ cf = reinterpret_cast<const double2*>(ev.coef) + ((int64_t)lk * ev.Kcp + tile * 16 + li) * 4;
        double cc = c0, ss = s0;
        for (int k = 0; k < ev.Kbp; k += 4) {
            // (loaded a step ahead by force: 595 instead of 587 us)
            const double2 x0 = cf[0], x1 = cf[1], x2 = cf[2], x3 = cf[3];
            cf += (int64_t)16 * ev.Kcp;
            acc[0] = __builtin_amdgcn_mfma_f64_16x16x4f64(cc, x0.x, acc[0], 0, 0, 0);
            acc[1] = __builtin_amdgcn_mfma_f64_16x16x4f64(cc, x0.y, acc[1], 0, 0, 0);
            acc[2] = __builtin_amdgcn_mfma_f64_16x16x4f64(cc, x1.x, acc[2], 0, 0, 0);
            acc[3] = __builtin_amdgcn_mfma_f64_16x16x4f64(cc, x1.y, acc[3], 0, 0, 0);
            acc[4] = __builtin_amdgcn_mfma_f64_16x16x4f64(cc, x2.x, acc[4], 0, 0, 0);
            acc[5] = __builtin_amdgcn_mfma_f64_16x16x4f64(cc, x2.y, acc[5], 0, 0, 0);
            acc[6] = __builtin_amdgcn_mfma_f64_16x16x4f64(cc, x3.x, acc[6], 0, 0, 0);
            acc[7] = __builtin_amdgcn_mfma_f64_16x16x4f64(cc, x3.y, acc[7], 0, 0, 0);
            const double cn = cc * c4 - ss * s4;
            ss = cc * s4 + ss * c4;
            cc = cn;
        }
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            // dpsi + i r_a psi of the low and the high face
            const double lr = acc[2][r] - ra[r] * acc[1][r], lm = acc[3][r] + ra[r] * acc[0][r];
            const double hr = acc[6][r] - ra[r] * acc[5][r], hm = acc[7][r] + ra[r] * acc[4][r];
            orr[r] += tc[r] * (w[r].x * (lr - hr) - w[r].y * (lm + hm));
            oi[r] += tc[r] * (w[r].x * (lm - hm) + w[r].y * (lr + hr));
            const double cn = tc[r] * c16[r] - ts[r] * s16[r];
            ts[r] = tc[r] * s16[r] + ts[r] * c16[r];
            tc[r] = cn;
        }
    }
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        for (int o = 8; o > 0; o >>= 1) {
            orr[r] += __shfl_xor(orr[r], o, 64);
            oi[r] += __shfl_xor(oi[r], o, 64);
        }
        const int64_t d = d0 + 4 * r + lk;
        if (li == 0 && d < nd) part[(int64_t)blockIdx.y * nd + d] = make_double2(orr[r], oi[r]);
    }
}

// out[d] = exp(-i r_hat . mid) times the rows of part, in order
__global__ void far_sum_kernel(const double3* __restrict__ dirs, int64_t nd, double3 mid,
                               const double2* __restrict__ part, int rows, double2* __restrict__ out) {
    const int64_t d = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (d >= nd) return;
    double2 s = part[d];
    for (int k = 1; k < rows; ++k) s = zadd(s, part[(int64_t)k * nd + d]);
    const double3 r = dirs[d];
    double sn, cs;
    sincos(-(r.x * mid.x + r.y * mid.y + r.z * mid.z), &sn, &cs);
    out[d] = zmul(s, make_double2(cs, sn));
}

// Directions with a component beyond 1 (no unit vector, but the formula holds
// for any): from the factors themselves.  A workgroup looks over `per` directions
// and takes those blocks of 16 that hold such a one, a block as the rows of products
// on the FP64 matrix cores: the factors g of an axis, folded with its transform to h
// = g W, then h_c P of the four planes of an axis's faces, and the sum over b with
// h_b and the faces' phases in the accumulators' lanes.  A block costs the same with
// one such direction as with 16.  Bound by the latency of the planes' loads (five
// per 16 products).  64 and 65160 such vectors: 64^3 0.14 and 1.28 ms, 160^3 0.49 and
// 6.6 ms (a workgroup per direction on the vector units: 5.0 and 79, 21 and 335 ms; the
// factors' products for every call, as it once was: 0.58 and 2.7, 1.4 and 7.3 ms).
constexpr double kFarLimit = 1.0 + 4.0e-16;
constexpr int kWideGroups = 256;  // workgroups at most, each with scratch of its own
constexpr int kWideWaves = 8;

struct FarWide {
    FarAxis ax[3];
    double pref[3];
    const double2* planes;  // phasors, [face][psi, dpsi][plane]
    const double2* tw;      // per axis exp(-2 pi i j / N)
    int longest;            // axis length
};

// scratch of one workgroup: h of the three axes, [index][direction], and g
__host__ __device__ inline int64_t wide_scratch(const FarWide& f) {
    return 16 * ((int64_t)f.ax[0].N + f.ax[1].N + f.ax[2].N + f.longest);
}

// c += a b, complex, on 16 x 16 x 4 tiles
__device__ __forceinline__ void zmfma(double2 a, double2 b, v4d& re, v4d& im) {
    re = __builtin_amdgcn_mfma_f64_16x16x4f64(a.x, b.x, re, 0, 0, 0);
    im = __builtin_amdgcn_mfma_f64_16x16x4f64(a.x, b.y, im, 0, 0, 0);
    re = __builtin_amdgcn_mfma_f64_16x16x4f64(-a.y, b.y, re, 0, 0, 0);
    im = __builtin_amdgcn_mfma_f64_16x16x4f64(a.y, b.x, im, 0, 0, 0);
}

__global__ __launch_bounds__(64 * kWideWaves) void far_wide_kernel(const double3* __restrict__ dirs, int64_t nd, int per,
                                                                   FarWide f, double2* scratch,
                                                                   double2* __restrict__ out) {
    __shared__ int todo[16];          // blocks of 16 that hold such a direction
    __shared__ double rr[3][16];      // the block's directions
    __shared__ double2 ph[6][16];     // pref times the phase of each face
    __shared__ double2 part[kWideWaves][16];
    constexpr int NT = 64 * kWideWaves;
    const int t = threadIdx.x, lane = t & 63, wave = t >> 6, li = lane & 15, lk = lane >> 4;
    const int64_t base = (int64_t)blockIdx.x * per;
    auto wide = [](double3 r) { return fabs(r.x) > kFarLimit || fabs(r.y) > kFarLimit || fabs(r.z) > kFarLimit; };
    if (t < 16) todo[t] = 0;
    __syncthreads();
    if (t < per && base + t < nd && wide(dirs[base + t])) todo[t >> 4] = 1;
    __syncthreads();
    double2* h = scratch + (int64_t)blockIdx.x * wide_scratch(f);
    double2* g = h + 16 * ((int64_t)f.ax[0].N + f.ax[1].N + f.ax[2].N);
    const int off[3] = {0, f.ax[0].N, f.ax[0].N + f.ax[1].N};
    for (int blk = 0; blk * 16 < per; ++blk) {
        if (!todo[blk]) continue;
        const int64_t d0 = base + blk * 16;
        __syncthreads();
        if (t < 16) {
            const double3 r = dirs[min(d0 + t, nd - 1)];
            const double v[3] = {r.x, r.y, r.z};
            for (int face = 0; face < 6; ++face) {
                const int a = face / 2, side = face % 2;
                double sn, cs;
                sincos(-v[a] * (f.ax[a].mid + (side ? f.ax[a].half : -f.ax[a].half)), &sn, &cs);
                const double w = side ? -f.pref[a] : f.pref[a];
                ph[face][t] = make_double2(w * cs, w * sn);
                rr[a][t] = v[a];
            }
        }
        __syncthreads();
        for (int a = 0; a < 3; ++a) {
            const int N = f.ax[a].N;
            for (int e = t; e < 16 * N; e += NT) g[e] = far_factor(f.ax[a], rr[a][e & 15], 0.0, e >> 4, false);
            __syncthreads();
            for (int j0 = wave * 16; j0 < N; j0 += 16 * kWideWaves) {
                const int j = j0 + li;
                v4d re = {0, 0, 0, 0}, im = {0, 0, 0, 0};
                int idx = (int)((int64_t)lk * j % N);
                const int hop = (int)((int64_t)4 * j % N);
                for (int k = lk; k - lk < N; k += 4) {
                    const double2 x = k < N ? g[k * 16 + li] : make_double2(0, 0);
                    zmfma(x, f.tw[off[a] + idx], re, im);
                    idx += hop;
                    if (idx >= N) idx -= N;
                }
#pragma unroll
                for (int r = 0; r < 4; ++r)
                    if (j < N) h[(int64_t)(off[a] + j) * 16 + 4 * r + lk] = make_double2(re[r], im[r]);
            }
            __syncthreads();
        }
        // tiles of 16 columns b of the three axes' planes, dealt to the waves
        double2 sum[4];
#pragma unroll
        for (int r = 0; r < 4; ++r) sum[r] = make_double2(0, 0);
        int job = 0;
        const double2* pl = f.planes;
        for (int a = 0; a < 3; ++a) {
            const int b = face_axis_b(a), c = face_axis_c(a);
            const int Nb = f.ax[b].N, Nc = f.ax[c].N;
            const int64_t np = (int64_t)Nb * Nc;
            const double2 *hb = h + (int64_t)off[b] * 16, *hc = h + (int64_t)off[c] * 16;
            for (int j0 = 0; j0 < Nb; j0 += 16, ++job) {
                if (job % kWideWaves != wave) continue;
                const int j = min(j0 + li, Nb - 1);
                v4d re[4], im[4];
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    re[q] = v4d{0, 0, 0, 0};
                    im[q] = v4d{0, 0, 0, 0};
                }
                for (int k = lk; k - lk < Nc; k += 4) {
                    const int kc = min(k, Nc - 1);
                    const double2 x = k < Nc ? hc[kc * 16 + li] : make_double2(0, 0);
                    const double2* y = pl + (int64_t)kc * Nb + j;
#pragma unroll
                    for (int q = 0; q < 4; ++q) zmfma(x, y[q * np], re[q], im[q]);
                }
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const int i = 4 * r + lk;
                    const double ra = rr[a][i];
                    // dpsi + i r_a psi of the low and the high face
                    const double2 lo = zmul(ph[2 * a][i], make_double2(re[1][r] - ra * im[0][r], im[1][r] + ra * re[0][r]));
                    const double2 hi = zmul(ph[2 * a + 1][i], make_double2(re[3][r] - ra * im[2][r], im[3][r] + ra * re[2][r]));
                    if (j0 + li < Nb) sum[r] = zadd(sum[r], zmul(hb[(int64_t)j * 16 + i], zadd(lo, hi)));
                }
            }
            pl += 4 * np;
        }
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            for (int o = 8; o > 0; o >>= 1) {
                sum[r].x += __shfl_xor(sum[r].x, o, 64);
                sum[r].y += __shfl_xor(sum[r].y, o, 64);
            }
            if (li == 0) part[wave][4 * r + lk] = sum[r];
        }
        __syncthreads();
        if (t < 16 && d0 + t < nd && wide(dirs[d0 + t])) {
            double2 s = part[0][t];
            for (int w = 1; w < kWideWaves; ++w) s = zadd(s, part[w][t]);
            out[d0 + t] = s;
        }
    }
}

// ---------------------------------------------------------------------------
// Fresnel points
// ---------------------------------------------------------------------------

constexpr int kNearThreads = 256;
constexpr int kNearPoints = 2;  // observation points per thread in near_kernel
constexpr int kCellChunk = 16;

struct FaceGeo {
    int a, b, c;
    int lo_b, lo_c, L, M;     // cell ranges
    double db, dc, xa;        // reduced spacings, face coordinate
    double xb0, xc0;          // first cell-centre coordinates
    double pref;
};

// Whether a point lies inside the box or is not finite (bit 0), and whether it
// is so far that its phases need the general sincos (bit 1)
__global__ void check_points_kernel(const double3* __restrict__ obs, int64_t n, double k0, double3 lo, double3 hi,
                                    double limit, unsigned* __restrict__ flags) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    unsigned f = 0;
    if (i < n) {
        const double3 o = obs[i];
        const double r[3] = {o.x * k0, o.y * k0, o.z * k0};
        const double l[3] = {lo.x, lo.y, lo.z}, h[3] = {hi.x, hi.y, hi.z};
        bool inside = true;
        for (int a = 0; a < 3; ++a) {
            if (!(r[a] > l[a] && r[a] < h[a])) inside = false;
            if (!isfinite(r[a])) inside = true;
        }
        f = (inside ? 1u : 0u) | (fabs(r[0]) > limit || fabs(r[1]) > limit || fabs(r[2]) > limit ? 2u : 0u);
    }
    if (f) atomicOr(flags, f);
}

// Share of the product of degrees (hp, hq) in the low term (p, q): e, its entry of E,
// times A^(hp - p) B^(hq - q)
__device__ __forceinline__ double econ_weight(double e, double A, double B, int p, int q, int hp, int hq) {
    for (int t = p; t < hp; ++t) e *= A;
    for (int t = hp; t < p; ++t) e /= A;
    for (int t = q; t < hq; ++t) e *= B;
    for (int t = hq; t < q; ++t) e /= B;
    return e;
}

// Economised terms Q[cell][field][low_row(p) + q], p + q <= 8, from the full
// products Qg[field][p][q][cell]: on the cells' disk (alpha_b / A)^2 +
// (alpha_c / B)^2 <= 1, A = d_b / 2, B = d_c / 2, a monomial of degree 9 to 16 is
// replaced by its least-squares polynomial of degree 8 (E, for the unit
// disk).  That leaves 1/11 to 1/32 of the largest value of a degree-9 monomial and
// 1/5 to 1/30 of one of degree 10 to 16.  Evaluated over the disk and all spectral
// indexes for 3 to 20 points per wavelength, A = B, the sums with E are within 1/35 of
// a^9 / 10!, the 9th-order term that the series drops (a = A), of those without, and
// their largest error against the exact sincs within 0.7 % of theirs (B = 0.6 A: 1.4 %
// below).  45 terms per field and cell instead of 81.
__global__ void economise_kernel(const double2* __restrict__ Qg, int64_t ncell, const double* __restrict__ E, double A,
                                 double Bs, double2* __restrict__ Q) {
    const int64_t id = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (id >= ncell * kLow * 2) return;
    const int64_t cell = id % ncell;
    const int k = (int)((id / ncell) % kLow), fld = (int)(id / (ncell * kLow));
    int p = 0;
    while (k >= low_row(p + 1)) ++p;
    const int q = k - low_row(p);
    const double2* g = Qg + (int64_t)fld * kPairs * ncell + cell;
    double2 s = g[(int64_t)(p * kTerms + q) * ncell];
    int h = 0;
    for (int hp = 1; hp < kTerms; ++hp)
        for (int hq = kTerms - hp; hq < kTerms; ++hq, ++h) {
            const double e = E[h * kLow + k];
            if (e == 0.0) continue;
            const double w = econ_weight(e, A, Bs, p, q, hp, hq);
            const double2 x = g[(int64_t)(hp * kTerms + hq) * ncell];
            s.x += w * x.x;
            s.y += w * x.y;
        }
    Q[(cell * 2 + fld) * kLow + k] = s;
}

// its adjoint: Qbar[field][p][q][cell] from the sums of the low terms
// low[field][k][cell]
__global__ void economise_adjoint_kernel(const double2* __restrict__ low, int64_t ncell, const double* __restrict__ E,
                                         double A, double Bs, double2* __restrict__ Qbar) {
    const int64_t id = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (id >= ncell * kPairs * 2) return;
    const int64_t cell = id % ncell;
    const int pq = (int)((id / ncell) % kPairs), fld = (int)(id / (ncell * kPairs));
    const int hp = pq / kTerms, hq = pq % kTerms;
    const double2* g = low + (int64_t)fld * kLow * ncell + cell;
    double2 s = make_double2(0, 0);
    if (hp + hq <= kOrder) {
        s = g[(int64_t)(low_row(hp) + hq) * ncell];
    } else {
        int h = 0;
        for (int t = 1; t < hp; ++t) h += t;   // row t holds the t pairs (t, 9 - t) .. (t, 8)
        h += hq - (kTerms - hp);
        for (int p = 0; p < kTerms; ++p)
            for (int q = 0; q + p < kTerms; ++q) {
                const int k = low_row(p) + q;
                const double e = E[h * kLow + k];
                if (e == 0.0) continue;
                const double w = econ_weight(e, A, Bs, p, q, hp, hq);
                const double2 x = g[(int64_t)k * ncell];
                s.x += w * x.x;
                s.y += w * x.y;
            }
    }
    Qbar[id] = s;
}

template <bool FAST>
__device__ __forceinline__ void phase(double x, double* sn, double* cs) {
    if constexpr (FAST) fast_sincos(x, sn, cs);
    else sincos(x, sn, cs);
}

// Q layout: [cell][field(0 psi, 1 dpsi)][low terms]
// One thread per K points; workgroup row blockIdx.y sums the cells
// [y * cells_per_split, (y + 1) * cells_per_split), so that few points still
// fill the chip.  Each row writes its partial sum (times the face prefactor)
// to part[y * n_obs + point]; add_splits_kernel adds the rows in order.
// K observation points per thread, kNearThreads apart (coalesced loads and
// stores): each coefficient read from LDS serves K points, which takes the
// kernel off the LDS read rate (one 16-byte broadcast per two FP64 FMAs
// with one point per thread; 306 VGPRs with four, 114 with two).  Bound by the FP64 vector rate: 216 FMAs of the
// two economised polynomials and about 80 instructions for the distance, its
// reciprocal and the phase per point and cell (360 and 170 with the 81-term
// products and the library's square root, division and sincos: 5.22 ms per
// face for 16384 points and 15876 cells, 2.39 ms now).
template <int K, bool FAST>
__global__ __launch_bounds__(kNearThreads) void near_kernel(const double3* __restrict__ obs, int64_t n_obs, double k0,
                                                            FaceGeo g, const double2* __restrict__ Q,
                                                            int64_t cells_per_split, double2* __restrict__ part) {
    __shared__ double2 sq[kCellChunk * 2 * kLow];
    bool live[K];
    bool any_live = false;
    double Ra[K], rb_[K], rc_[K];  // point in the face frame (normal, b, c)
    double2 acc[K];
#pragma unroll
    for (int k = 0; k < K; ++k) {
        const int64_t pi = ((int64_t)blockIdx.x * K + k) * kNearThreads + threadIdx.x;
        live[k] = pi < n_obs;
        any_live |= live[k];
        // an idle slot gets a point one unit off the face, so that its
        // (discarded) sums stay finite
        double ra = g.xa + 1.0, rb = 0, rc = 0;
        if (live[k]) {
            const double3 o = obs[pi];
            const double x = o.x * k0, y = o.y * k0, z = o.z * k0;
            ra = g.a == 0 ? x : g.a == 1 ? y : z;
            rb = g.b == 0 ? x : g.b == 1 ? y : z;
            rc = g.c == 0 ? x : g.c == 1 ? y : z;
        }
        Ra[k] = ra - g.xa;
        rb_[k] = rb;
        rc_[k] = rc;
        acc[k] = make_double2(0, 0);
    }
    const double hb = 0.5 * g.db, hc = 0.5 * g.dc;
    const int64_t ncell = (int64_t)g.L * g.M;
    const int64_t c_lo = (int64_t)blockIdx.y * cells_per_split;
    const int64_t c_hi = min<int64_t>(ncell, c_lo + cells_per_split);
    constexpr int per_cell = 2 * kLow;
    for (int64_t c0 = c_lo; c0 < c_hi; c0 += kCellChunk) {
        const int nc = (int)min<int64_t>(kCellChunk, c_hi - c0);
        __syncthreads();
        for (int e = threadIdx.x; e < nc * per_cell; e += kNearThreads) sq[e] = Q[c0 * per_cell + e];
        __syncthreads();
        if (!any_live) continue;
#pragma unroll 1
        for (int ci = 0; ci < nc; ++ci) {
            const int cell = (int)(c0 + ci);
            const int m = cell / g.L, l = cell - m * g.L;
            double Rn[K], inv[K], ab[K], ac[K];
#pragma unroll
            for (int k = 0; k < K; ++k) {
                const double Rb = rb_[k] - (g.xb0 + l * g.db);
                const double Rc = rc_[k] - (g.xc0 + m * g.dc);
                sqrt_rsqrt(Ra[k] * Ra[k] + Rb * Rb + Rc * Rc, &Rn[k], &inv[k]);
                ab[k] = hb * Rb * inv[k];
                ac[k] = hc * Rc * inv[k];
            }
            const double2* q = &sq[ci * per_cell];
            double2 S0[K], S1[K];
#pragma unroll 1
            for (int fld = 0; fld < 2; ++fld) {
                double2 outer[K];
#pragma unroll
                for (int k = 0; k < K; ++k) outer[k] = make_double2(0, 0);
#pragma unroll
                for (int p = kOrder; p >= 0; --p) {
                    const double2* row = q + fld * kLow + low_row(p);
                    double2 inner[K];
                    const double2 top = row[kOrder - p];
#pragma unroll
                    for (int k = 0; k < K; ++k) inner[k] = top;
#pragma unroll
                    for (int qq = kOrder - p - 1; qq >= 0; --qq) {
                        const double2 cq = row[qq];
#pragma unroll
                        for (int k = 0; k < K; ++k) {
                            inner[k].x = fma(inner[k].x, ac[k], cq.x);
                            inner[k].y = fma(inner[k].y, ac[k], cq.y);
                        }
                    }
#pragma unroll
                    for (int k = 0; k < K; ++k) {
                        outer[k].x = fma(outer[k].x, ab[k], inner[k].x);
                        outer[k].y = fma(outer[k].y, ab[k], inner[k].y);
                    }
                }
#pragma unroll
                for (int k = 0; k < K; ++k) {
                    if (fld == 0) S0[k] = outer[k];
                    else S1[k] = outer[k];
                }
            }
            // e^{iR}/R (S_dpsi + (i - 1/R) (R_a/R) S_psi)
#pragma unroll
            for (int k = 0; k < K; ++k) {
                const double ra = Ra[k] * inv[k];
                const double2 coef = make_double2(-inv[k] * ra, ra);
                const double2 inner = zadd(S1[k], zmul(coef, S0[k]));
                double sn, cs;
                phase<FAST>(Rn[k], &sn, &cs);
                acc[k] = zadd(acc[k], zmul(make_double2(cs * inv[k], sn * inv[k]), inner));
            }
        }
    }
#pragma unroll
    for (int k = 0; k < K; ++k) {
        const int64_t pi = ((int64_t)blockIdx.x * K + k) * kNearThreads + threadIdx.x;
        if (live[k]) part[(int64_t)blockIdx.y * n_obs + pi] = make_double2(acc[k].x * g.pref, acc[k].y * g.pref);
    }
}

// out[i] (+)= sum over the split rows k = 0, 1, ... of part[k * n + i], in
// row order
__global__ void add_splits_kernel(const double2* __restrict__ part, int splits, int64_t n, bool accumulate,
                                  double2* __restrict__ out) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    double2 acc = part[i];
    for (int k = 1; k < splits; ++k) acc = zadd(acc, part[(int64_t)k * n + i]);
    out[i] = accumulate ? zadd(out[i], acc) : acc;
}

// Adjoint of the per-point cell sums: for one cell and the low terms (p, q),
// low[fld][k][cell] = sum_o conj(pref e^{iR}/R alpha_b^p alpha_c^q [coef]) g_o,
// coef = (i - 1/R) R_a / R for the psi field (fld 0), 1 for dpsi (fld 1).
constexpr int kAdjObsChunk = 256;
constexpr int kAdjGroups = 3;

// Workgroup row blockIdx.y sums the points [y * obs_per_split, (y + 1) *
// obs_per_split) into its own copy of low (+ y * 2 kLow ncell);
// add_splits_kernel adds the copies in order.  One thread per (cell, group
// of 15 terms): rows p of lengths 9 - p in three groups of equal size, {0, 3},
// {1, 2}, {4, 5, 6, 7, 8}, so that the distance and the phase of a (cell,
// point) pair serve 15 terms of both fields and the sums stay in registers.
template <int G, bool FAST>
__device__ __forceinline__ void near_adjoint_group(const double3* __restrict__ obs, const double2* __restrict__ gv,
                                                   int64_t n_obs, double k0, const FaceGeo& g, int64_t obs_per_split,
                                                   double3* so, double2* sg, double2* __restrict__ low) {
    constexpr int rows[3][5] = {{0, 3, -1, -1, -1}, {1, 2, -1, -1, -1}, {4, 5, 6, 7, 8}};
    constexpr int nrows = G == 2 ? 5 : 2;
    constexpr int kPer = kLow / kAdjGroups;
    const int64_t ncell = (int64_t)g.L * g.M;
    const int64_t cell_ = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const bool live = cell_ < ncell;
    const int64_t cell = live ? cell_ : 0;
    const int m = (int)(cell / g.L), l = (int)(cell % g.L);
    const double yb = g.xb0 + l * g.db, yc = g.xc0 + m * g.dc;
    const double hb = 0.5 * g.db, hc = 0.5 * g.dc;
    double2 acc[2][kPer];
#pragma unroll
    for (int i = 0; i < kPer; ++i) acc[0][i] = acc[1][i] = make_double2(0, 0);
    const int64_t o_lo = (int64_t)blockIdx.y * obs_per_split;
    const int64_t o_hi = min<int64_t>(n_obs, o_lo + obs_per_split);
    for (int64_t o0 = o_lo; o0 < o_hi; o0 += kAdjObsChunk) {
        const int no = (int)min<int64_t>(kAdjObsChunk, o_hi - o0);
        __syncthreads();
        for (int e = threadIdx.x; e < no; e += blockDim.x) {
            so[e] = obs[o0 + e];
            sg[e] = gv[o0 + e];
        }
        __syncthreads();
        if (!live) continue;
#pragma unroll 1
        for (int e = 0; e < no; ++e) {
            const double x = so[e].x * k0, y = so[e].y * k0, z = so[e].z * k0;
            const double Ra = (g.a == 0 ? x : g.a == 1 ? y : z) - g.xa;
            const double Rb = (g.b == 0 ? x : g.b == 1 ? y : z) - yb;
            const double Rc = (g.c == 0 ? x : g.c == 1 ? y : z) - yc;
            double Rn, inv;
            sqrt_rsqrt(Ra * Ra + Rb * Rb + Rc * Rc, &Rn, &inv);
            const double ab = hb * Rb * inv, ac = hc * Rc * inv;
            double sn, cs;
            phase<FAST>(Rn, &sn, &cs);
            const double2 gg = sg[e];
            const double rr = Ra * inv;
            // conj(pref e^{iR}/R) g and conj(coef) = (-i - 1/R) R_a/R times it
            const double wr = g.pref * inv;
            const double2 b1 = make_double2(wr * (cs * gg.x + sn * gg.y), wr * (cs * gg.y - sn * gg.x));
            const double2 b0 = make_double2(-inv * rr * b1.x + rr * b1.y, -inv * rr * b1.y - rr * b1.x);
            double abp = 1.0;
            int at = 0;
#pragma unroll
            for (int i = 0; i < nrows; ++i) {
                const int p = rows[G][i];
#pragma unroll
                for (int t = (i ? rows[G][i - 1] : 0); t < p; ++t) abp *= ab;
                double w = abp;
#pragma unroll
                for (int q = 0; q < kTerms - p; ++q, ++at) {
                    acc[0][at].x = fma(w, b0.x, acc[0][at].x);
                    acc[0][at].y = fma(w, b0.y, acc[0][at].y);
                    acc[1][at].x = fma(w, b1.x, acc[1][at].x);
                    acc[1][at].y = fma(w, b1.y, acc[1][at].y);
                    w *= ac;
                }
            }
        }
    }
    if (!live) return;
    double2* __restrict__ dst = low + (int64_t)blockIdx.y * 2 * kLow * ncell;
    int at = 0;
#pragma unroll
    for (int i = 0; i < nrows; ++i) {
        const int p = rows[G][i];
#pragma unroll
        for (int q = 0; q < kTerms - p; ++q, ++at)
            for (int f = 0; f < 2; ++f) dst[((int64_t)f * kLow + low_row(p) + q) * ncell + cell] = acc[f][at];
    }
}

template <bool FAST>
__global__ __launch_bounds__(128) void near_adjoint_kernel(const double3* __restrict__ obs, const double2* __restrict__ gv,
                                                           int64_t n_obs, double k0, FaceGeo g, int64_t obs_per_split,
                                                           double2* __restrict__ low) {
    __shared__ double3 so[kAdjObsChunk];
    __shared__ double2 sg[kAdjObsChunk];
    if (blockIdx.z == 0) near_adjoint_group<0, FAST>(obs, gv, n_obs, k0, g, obs_per_split, so, sg, low);
    else if (blockIdx.z == 1) near_adjoint_group<1, FAST>(obs, gv, n_obs, k0, g, obs_per_split, so, sg, low);
    else near_adjoint_group<2, FAST>(obs, gv, n_obs, k0, g, obs_per_split, so, sg, low);
}

// out = conj(sum of the 9 planes x[p]) * scale as complex64
__global__ void conj_scale_kernel(const double2* __restrict__ x, int64_t n, double scale, float2* __restrict__ out) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    double2 s = x[i];
    for (int p = 1; p < kTerms; ++p) s = zadd(s, x[p * n + i]);
    out[i] = make_float2((float)(s.x * scale), (float)(-s.y * scale));
}

// X[t][l][m]: the expansion of the cell integral along one axis (`cells` cells
// from grid index lo, FFT length N): for cell l and spectral index m (signed
// m') the Taylor coefficient t of the sinc factor (tay[t][m]) times the phase of the
// cell centre
__global__ void expansion_kernel(const double* __restrict__ tay, int N, int lo, int cells, double2* __restrict__ X) {
    const int64_t id = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (id >= (int64_t)kTerms * cells * N) return;
    const int m = (int)(id % N), l = (int)((id / N) % cells), t = (int)(id / ((int64_t)N * cells));
    const int bp = m < N / 2 ? m : m - N;
    // 2 pi b' x_l / (N d), x_l = (lo + l - N/2 + 1/2) d, in half turns over N
    const int64_t turns = ((int64_t)bp * (2 * (lo + l) - N + 1)) % (2 * N);
    double sn, cs;
    sincospi((double)turns / N, &sn, &cs);
    const double w = ((bp & 1) ? -1.0 : 1.0) * tay[(int64_t)t * N + m];
    X[id] = make_double2(w * cs, w * sn);
}

// sinc(x - alpha) = sum_p s_p(x) alpha^p, s_p = (-1)^p sinc^(p)(x)/p!
void sinc_taylor(double x, double* s) {
    for (int p = 0; p <= kOrder; ++p) {
        double acc = 0.0;
        for (int j = 0; j < 40; ++j) {
            if (2 * j < p) continue;
            // (-1)^j (2j)! / ((2j-p)! (2j+1)!) x^(2j-p)
            double c = (j & 1) ? -1.0 : 1.0;
            for (int t = 2 * j - p + 1; t <= 2 * j; ++t) c *= t;
            for (int t = 2; t <= 2 * j + 1; ++t) c /= t;
            acc += c * std::pow(x, 2 * j - p);
        }
        double fact = 1.0;
        for (int t = 2; t <= p; ++t) fact *= t;
        s[p] = ((p & 1) ? -1.0 : 1.0) * acc / fact;
    }
}

// Least-squares polynomials of total degree <= 8 on the unit disk of the 36
// monomials u^p v^q, 9 <= p + q, p, q <= 8, with the Chebyshev weight
// 1 / sqrt(1 - r^2): E[h][low_row(p') + q'], h counting (p, q) row by row.  By
// parity only p' = p, q' = q (mod 2) occur.  Modified Gram-Schmidt on a product
// grid of the disk, in long double.
const std::vector<double>& economisation() {
    static const std::vector<double> table = [] {
        constexpr int nr = 24, na = 64;
        std::vector<double> E((size_t)kHigh * kLow, 0.0);
        std::vector<long double> u, v;
        for (int i = 0; i < nr; ++i)
            for (int j = 0; j < na; ++j) {
                // r dr / sqrt(1 - r^2): 1 - r^2 = t^2, t uniform (Gauss-Legendre not needed: midpoints)
                const long double t = (i + 0.5L) / nr, r = std::sqrt(1.0L - t * t), f = 2.0L * 3.14159265358979323846264L * (j + 0.5L) / na;
                u.push_back(r * std::cos(f));
                v.push_back(r * std::sin(f));
            }
        const size_t S = u.size();
        auto column = [&](int p, int q) {
            std::vector<long double> c(S);
            for (size_t s = 0; s < S; ++s) {
                long double x = 1;
                for (int t = 0; t < p; ++t) x *= u[s];
                for (int t = 0; t < q; ++t) x *= v[s];
                c[s] = x;
            }
            return c;
        };
        for (int par = 0; par < 4; ++par) {
            // orthonormal columns and the triangular factor of this parity's low monomials
            std::vector<int> idx;
            std::vector<std::vector<long double>> Q, R;
            for (int p = par & 1; p < kTerms; p += 2)
                for (int q = par >> 1; p + q < kTerms; q += 2) {
                    std::vector<long double> c = column(p, q), r(Q.size() + 1, 0.0L);
                    for (int pass = 0; pass < 2; ++pass)
                        for (size_t j = 0; j < Q.size(); ++j) {
                            long double d = 0;
                            for (size_t s = 0; s < S; ++s) d += Q[j][s] * c[s];
                            for (size_t s = 0; s < S; ++s) c[s] -= d * Q[j][s];
                            r[j] += d;
                        }
                    long double n = 0;
                    for (size_t s = 0; s < S; ++s) n += c[s] * c[s];
                    n = std::sqrt(n);
                    for (size_t s = 0; s < S; ++s) c[s] /= n;
                    r[Q.size()] = n;
                    Q.push_back(c);
                    R.push_back(r);
                    idx.push_back(low_row(p) + q);
                }
            int h = 0;
            for (int hp = 1; hp < kTerms; ++hp)
                for (int hq = kTerms - hp; hq < kTerms; ++hq, ++h) {
                    if ((hp & 1) != (par & 1) || (hq & 1) != (par >> 1)) continue;
                    std::vector<long double> c = column(hp, hq), d(Q.size());
                    for (size_t j = 0; j < Q.size(); ++j) {
                        d[j] = 0;
                        for (size_t s = 0; s < S; ++s) d[j] += Q[j][s] * c[s];
                        for (size_t s = 0; s < S; ++s) c[s] -= d[j] * Q[j][s];
                    }
                    // back substitution: R x = d, R[j][i] the coefficient of q_i in column j
                    for (size_t j = Q.size(); j-- > 0;) {
                        long double x = d[j];
                        for (size_t i = j + 1; i < Q.size(); ++i) x -= R[i][j] * d[i];
                        d[j] = x / R[j][j];
                    }
                    for (size_t j = 0; j < Q.size(); ++j) E[(size_t)h * kLow + idx[j]] = (double)d[j];
                }
        }
        return E;
    }();
    return table;
}

// Chebyshev terms of a function of exponential type X on [-1, 1] (the
// coefficients are Bessel functions J_k(X) of the phases' amplitudes): the
// first k past X with 2 |J_k(X)| < 2^-57
int far_terms(double X) {
    int k = (int)X + 2;
    // J_k(X) <= (e X / 2 k)^k / sqrt(2 pi k), which falls monotonically past X e / 2;
    // below that J_k(X) ~ Ai-like decay: the uniform bound exp(-k (w - tanh w)), cosh w = k / X
    for (;; ++k) {
        const double w = std::acosh(k / X);
        const double lg = -k * (w - std::tanh(w)) - 0.5 * std::log(2 * kPi * k * std::tanh(w));
        if (lg + std::log(2.0) < -57 * std::log(2.0)) break;
    }
    return k + 1;
}

}  // namespace

struct ProjectState {
    double2* phasors = nullptr;   // [face][2][plane]
    double2* work = nullptr;      // scratch
    size_t work_bytes = 0;
    double2* part = nullptr;      // per-split partial sums of the point kernels
    size_t part_bytes = 0;
    double2* low = nullptr;       // adjoint: the splits' sums
    size_t low_bytes = 0;
    unsigned* flags = nullptr;    // check_points_kernel's result
    // tables, built on first use (they depend on the grid and the box only),
    // each with the plane DFT folded in
    double2* near_tab = nullptr;  // per axis [t][cell][N]: sinc-Taylor expansion of the cell integral
    double* econ = nullptr;       // economisation table
    double2* far_tab = nullptr;   // per axis [K][N]: Chebyshev coefficients of the far factor
    // the far field's scratch, behind the tables: of one size for any number of
    // directions and its own, so that a far field captured by a caller finds it and no
    // later call moves it
    double2* far_work = nullptr;  // coefficients, products, far_wide_kernel's scratch
    double2* far_part = nullptr;  // [rows][direction]: far_eval_kernel's sums
    int64_t near_off[4] = {0, 0, 0, 0};
    int64_t far_off[4] = {0, 0, 0, 0};
    int K[3] = {0, 0, 0};
    int64_t coef_off[4] = {0, 0, 0, 0}, far_y = 0, far_c = 0;  // in far_work
    FarWide wide{};
    int64_t face_off[7] = {0, 0, 0, 0, 0, 0, 0};
    int64_t total = 0;
};

namespace {

template <class T>
hipError_t ensure(T** ptr, size_t* have, size_t need) {
    if (*have >= need) return hipSuccess;
    if (*ptr) {
        (void)hipDeviceSynchronize();  // queued launches may still use the old buffer
        (void)hipFree(*ptr);
    }
    *ptr = nullptr;
    *have = 0;
    hipError_t e = hipMalloc((void**)ptr, need);
    if (e == hipSuccess) *have = need;
    return e;
}

// Rows of workgroups a point kernel is split into: enough for about eight
// waves per SIMD (256 CUs x 4 SIMDs) when the points alone give fewer, at
// most `cap` (the number of independent pieces of the summed range)
constexpr int64_t kTargetWaves = 8 * 1024;
int split_count(int64_t waves, int64_t cap) {
    int64_t k = (kTargetWaves + waves - 1) / std::max<int64_t>(waves, 1);
    k = std::min<int64_t>(k, std::min<int64_t>(cap, 64));
    return (int)std::max<int64_t>(k, 1);
}

unsigned blocks_of(int64_t n, int per = 256) { return (unsigned)((n + per - 1) / per); }

#define TRY(x)                                \
    do {                                      \
        hipError_t _e = (x);                  \
        if (_e != hipSuccess) return _e;      \
    } while (0)

// the projection's state and the normalised phasors of this call
hipError_t prepare(ProjectState** pst, const pstd_problem& p, double2* const acc[3], const int64_t points[3],
                   PhasorScale scale, hipStream_t stream) {
    if (!*pst) {
        ProjectState* s = new ProjectState();
        int64_t off = 0;
        for (int f = 0; f < 6; ++f) {
            s->face_off[f] = off;
            off += 2 * points[f / 2];
        }
        s->face_off[6] = off;
        s->total = off;
        hipError_t e;
        if ((e = hipMalloc(&s->phasors, off * sizeof(double2))) || (e = hipMalloc(&s->flags, sizeof(unsigned)))) {
            project_free(s);
            return e;
        }
        *pst = s;
    }
    return finalize_phasors(acc, points, scale, (*pst)->phasors, stream);
}

}  // namespace

hipError_t finalize_phasors(double2* const acc[3], const int64_t points[3], PhasorScale scale, double2* out,
                            hipStream_t stream) {
    FinalizeArgs f{};
    int blocks = 0;
    for (int a = 0; a < 3; ++a) {
        f.acc[a] = acc[a];
        f.points[a] = points[a];
        f.blocks[a] = (int)blocks_of(points[a]);
        blocks += 2 * f.blocks[a];
    }
    hipLaunchKernelGGL(finalize_kernel, dim3(blocks), dim3(256), 0, stream, f, scale.v, scale.d, out);
    return hipGetLastError();
}

namespace {

int cells_of(const pstd_problem& p, int a) { return p.surf_hi[a] - p.surf_lo[a]; }

FarAxis far_axis(const pstd_problem& p, const double dxb[3], int a) {
    FarAxis x;
    x.N = p.n[a];
    x.lo = p.surf_lo[a];
    x.hi = p.surf_hi[a];
    x.d = dxb[a];
    x.mid = dxb[a] * (0.5 * (x.lo + x.hi) - x.N / 2);
    x.half = dxb[a] * 0.5 * (x.hi - x.lo);
    return x;
}

// The near tables of the three axes in one device array: per axis [t][cell][N],
// the transform of a plane line folded in (X W)
hipError_t near_tables(ProjectState* s, const pstd_problem& p, hipStream_t stream) {
    if (s->near_tab) return hipSuccess;
    int64_t total = 0;
    size_t work = 0;
    for (int a = 0; a < 3; ++a) {
        const int64_t N = p.n[a], rows = (int64_t)kTerms * cells_of(p, a);
        s->near_off[a] = total;
        total += rows * N;
        work = std::max(work, (size_t)(rows * N + N * N) * sizeof(double2) + (size_t)kTerms * N * sizeof(double));
    }
    const std::vector<double>& E = economisation();
    TRY(ensure(&s->work, &s->work_bytes, work));
    double2* tab = nullptr;
    double* econ = nullptr;
    auto undo = [&](hipError_t e) {
        (void)hipStreamSynchronize(stream);
        (void)hipFree(tab);
        (void)hipFree(econ);
        return e;
    };
    hipError_t e;
    if ((e = hipMalloc(&tab, (size_t)total * sizeof(double2))) || (e = hipMalloc(&econ, E.size() * sizeof(double))) ||
        (e = hipMemcpy(econ, E.data(), E.size() * sizeof(double), hipMemcpyHostToDevice)))
        return undo(e);
    for (int a = 0; a < 3; ++a) {
        const int N = p.n[a], cells = cells_of(p, a);
        const int64_t rows = (int64_t)kTerms * cells;
        std::vector<double> tay((size_t)kTerms * N);
        for (int m = 0; m < N; ++m) {
            double sp[kTerms];
            sinc_taylor(kPi * (m < N / 2 ? m : m - N) / N, sp);
            for (int t = 0; t < kTerms; ++t) tay[(size_t)t * N + m] = sp[t];
        }
        double2* X = s->work;
        double2* W = X + rows * N;
        double* dtay = reinterpret_cast<double*>(W + (int64_t)N * N);
        // the scratch is the previous axis's until its products are done
        if ((e = hipStreamSynchronize(stream)) ||
            (e = hipMemcpy(dtay, tay.data(), tay.size() * sizeof(double), hipMemcpyHostToDevice)))
            return undo(e);
        hipLaunchKernelGGL(dft_matrix_kernel, dim3(blocks_of((int64_t)N * N)), dim3(256), 0, stream, N, W);
        hipLaunchKernelGGL(expansion_kernel, dim3(blocks_of(rows * N)), dim3(256), 0, stream, dtay, N, p.surf_lo[a],
                           cells, X);
        if ((e = zgemm((int)rows, N, N, ZOp{X, N}, ZOp{W, N}, tab + s->near_off[a], N, 0, 0, 1, 1, {}, stream)))
            return undo(e);
    }
    s->near_tab = tab;
    s->econ = econ;
    return hipSuccess;
}

// Directions of one launch, and the values of far_part: rows of a launch are 3
// jsplit, jsplit at most the waves that 2048 lack, so rows times directions stay
// under 3 kFarChunk + 2048 * 16
constexpr int64_t kFarChunk = 1 << 16;
static_assert(kFarChunk <= 256 * kWideGroups, "a workgroup of far_wide_kernel looks over 256 directions at most");
constexpr int64_t kFarPart = 3 * kFarChunk + 2048 * 16;

int far_kbp(const ProjectState* s, int a) { return (s->K[face_axis_b(a)] + 3) / 4 * 4; }
int far_kcp(const ProjectState* s, int a) { return (s->K[face_axis_c(a)] + 15) / 16 * 16; }

// The far tables of the three axes, per axis [K][N]: the Chebyshev coefficients of
// the centred factor with the transform folded in (D G W); and the far field's
// scratch, in the same allocation.  Nothing after the first call.
hipError_t far_tables(ProjectState* s, const pstd_problem& p, const double dxb[3], hipStream_t stream) {
    if (s->far_tab) return hipSuccess;
    // host values: the Chebyshev nodes, twiddles exp(-2 pi i j / N)
    constexpr long double kPiL = 3.14159265358979323846264L;
    std::vector<double2> host;
    int64_t total = 0, build = 0, node_off[3];
    FarWide fw{};
    for (int a = 0; a < 3; ++a) {
        const int b = face_axis_b(a), c = face_axis_c(a);
        fw.ax[a] = far_axis(p, dxb, a);
        fw.longest = std::max(fw.longest, fw.ax[a].N);
        fw.pref[a] = dxb[b] * dxb[c] / (4 * kPi * p.n[b] * p.n[c]) / p.k0;
        const int64_t N = p.n[a], K = s->K[a] = far_terms(fw.ax[a].half);
        s->far_off[a] = total;
        total += K * N;
        build = std::max(build, 2 * K * N + K * K + N * N);
        for (int j = 0; j < N; ++j) {
            const long double x = 2 * kPiL * j / N;
            host.push_back(make_double2((double)std::cos(x), (double)-std::sin(x)));
        }
    }
    for (int a = 0; a < 3; ++a) {
        node_off[a] = (int64_t)host.size();
        for (int64_t j = 0; j < s->K[a]; ++j) {
            const long double r = std::cos(kPiL * (j + 0.5L) / s->K[a]);
            host.push_back(make_double2((double)r, (double)(r - (double)r)));
        }
    }
    s->far_y = s->far_c = 0;
    for (int a = 0; a < 3; ++a) {
        const int b = face_axis_b(a), c = face_axis_c(a);
        s->coef_off[a + 1] = s->coef_off[a] + (int64_t)far_kbp(s, a) * far_kcp(s, a) * 4;
        s->far_y = std::max(s->far_y, (int64_t)4 * p.n[c] * s->K[b]);
        s->far_c = std::max(s->far_c, (int64_t)4 * s->K[c] * s->K[b]);
    }
    // (the tables are built in the scratch)
    const int64_t work = std::max(build, s->coef_off[3] + s->far_y + s->far_c + kWideGroups * wide_scratch(fw));
    double2* tab = nullptr;
    hipError_t e = hipMalloc(&tab, (size_t)(total + (int64_t)host.size() + work + kFarPart) * sizeof(double2));
    double2* vals = tab + total;
    double2* scratch = vals + host.size();
    if (!e) e = hipMemcpy(vals, host.data(), host.size() * sizeof(double2), hipMemcpyHostToDevice);
    for (int a = 0; a < 3 && !e; ++a) {
        const int N = p.n[a], K = s->K[a];
        double2* G = scratch;
        double2* DG = G + (int64_t)K * N;
        double2* D = DG + (int64_t)K * N;
        double2* W = D + (int64_t)K * K;
        hipLaunchKernelGGL(far_nodes_kernel, dim3(blocks_of((int64_t)K * N)), dim3(256), 0, stream, fw.ax[a], K,
                           vals + node_off[a], G);
        hipLaunchKernelGGL(far_dct_kernel, dim3(blocks_of((int64_t)K * K)), dim3(256), 0, stream, K, D);
        hipLaunchKernelGGL(dft_matrix_kernel, dim3(blocks_of((int64_t)N * N)), dim3(256), 0, stream, N, W);
        e = zgemm(K, N, K, ZOp{D, K}, ZOp{G, N}, DG, N, 0, 0, 1, 1, {}, stream);
        if (!e) e = zgemm(K, N, N, ZOp{DG, N}, ZOp{W, N}, tab + s->far_off[a], N, 0, 0, 1, 1, {}, stream);
    }
    if (e) {
        (void)hipStreamSynchronize(stream);
        (void)hipFree(tab);
        return e;
    }
    fw.tw = vals;
    fw.planes = s->phasors;
    s->wide = fw;
    s->far_tab = tab;
    s->far_work = scratch;
    s->far_part = scratch + work;
    return hipSuccess;
}

FaceGeo face_geo(const pstd_problem& p, const double dxb[3], int f) {
    FaceGeo g;
    const int a = f / 2, side = f % 2, b = face_axis_b(a), c = face_axis_c(a);
    g.a = a;
    g.b = b;
    g.c = c;
    g.lo_b = p.surf_lo[b];
    g.lo_c = p.surf_lo[c];
    g.L = cells_of(p, b);
    g.M = cells_of(p, c);
    g.db = dxb[b];
    g.dc = dxb[c];
    g.xa = ((side == 0 ? p.surf_lo[a] : p.surf_hi[a]) - p.n[a] / 2) * dxb[a];
    g.xb0 = (p.surf_lo[b] - p.n[b] / 2 + 0.5) * dxb[b];
    g.xc0 = (p.surf_lo[c] - p.n[c] / 2 + 0.5) * dxb[c];
    g.pref = (side == 0 ? 1.0 : -1.0) * dxb[b] * dxb[c] / (4 * kPi * p.n[b] * p.n[c]);
    return g;
}

// the largest coordinate of a point whose distances to the box stay within
// fast_sincos's range
double fast_limit(const pstd_problem& p, const double dxb[3]) {
    double box = 0;
    for (int a = 0; a < 3; ++a) box = std::max(box, dxb[a] * p.n[a]);
    return kFastSincosLimit / 2 - box;
}

// flags of the observation points (see check_points_kernel), read back
hipError_t check_points(ProjectState* s, const pstd_problem& p, const double dxb[3], const double3* obs, int64_t n_obs,
                        unsigned* flags, hipStream_t stream) {
    double lo[3], hi[3];
    for (int a = 0; a < 3; ++a) {
        lo[a] = (p.surf_lo[a] - p.n[a] / 2) * dxb[a];
        hi[a] = (p.surf_hi[a] - p.n[a] / 2) * dxb[a];
    }
    TRY(hipMemsetAsync(s->flags, 0, sizeof(unsigned), stream));
    hipLaunchKernelGGL(check_points_kernel, dim3(blocks_of(n_obs)), dim3(256), 0, stream, obs, n_obs, p.k0,
                       make_double3(lo[0], lo[1], lo[2]), make_double3(hi[0], hi[1], hi[2]), fast_limit(p, dxb), s->flags);
    TRY(hipGetLastError());
    TRY(hipMemcpyAsync(flags, s->flags, sizeof(unsigned), hipMemcpyDeviceToHost, stream));
    return hipStreamSynchronize(stream);
}

}  // namespace

hipError_t far_field(ProjectState** pst, const pstd_problem& p, const double dxb[3], double2* const acc[3],
                     const int64_t points[3], PhasorScale scale, const double3* dirs, int64_t n_dir, double2* out,
                     hipStream_t stream, std::string* msg) {
    // a caller's capture allows no allocation: refused before anything is done,
    // unless an earlier call (far field or points) has made the tables
    if (stream_capturing(stream) && !(*pst && (*pst)->far_tab)) return hipErrorStreamCaptureUnsupported;
    TRY(prepare(pst, p, acc, points, scale, stream));
    ProjectState* s = *pst;
    TRY(far_tables(s, p, dxb, stream));
    // coefficients of every axis's two faces: C = B_c P B_b^T
    const int64_t* coef_off = s->coef_off;
    int Kbp[3], Kcp[3];
    for (int a = 0; a < 3; ++a) {
        Kbp[a] = far_kbp(s, a);
        Kcp[a] = far_kcp(s, a);
    }
    double2* coef = s->far_work;
    double2* Y = coef + coef_off[3];
    double2* C = Y + s->far_y;
    double2* scratch = C + s->far_c;
    FarArgs args{};
    const FarWide& fw = s->wide;
    double mid[3];
    for (int a = 0; a < 3; ++a) {
        const int b = face_axis_b(a), c = face_axis_c(a);
        const int Nb = p.n[b], Nc = p.n[c], Kb = s->K[b], Kc = s->K[c];
        const int64_t np = (int64_t)Nb * Nc;
        // the four planes (low psi, low dpsi, high psi, high dpsi) lie side by side
        TRY(zgemm(Nc, Kb, Nb, ZOp{s->phasors + s->face_off[2 * a], Nb, np}, ZOp{s->far_tab + s->far_off[b], Nb}, Y, Kb,
                  (int64_t)Nc * Kb, 0, 4, 1, ZOpts{false, false, true, false}, stream));
        TRY(zgemm(Kc, Kb, Nc, ZOp{s->far_tab + s->far_off[c], Nc}, ZOp{Y, Kb, (int64_t)Nc * Kb}, C, Kb,
                  (int64_t)Kc * Kb, 0, 4, 1, {}, stream));
        const int64_t n = (int64_t)Kbp[a] * Kcp[a] * 4;
        hipLaunchKernelGGL(far_pack_kernel, dim3(blocks_of(n)), dim3(256), 0, stream, Kb, Kc, Kbp[a], Kcp[a], C,
                           coef + coef_off[a]);
        args.ax[a] = FarEval{reinterpret_cast<const double*>(coef + coef_off[a]), Kbp[a], Kcp[a], fw.ax[a].half,
                             std::fma(0.5 * dxb[a], p.surf_hi[a] - p.surf_lo[a], -fw.ax[a].half), fw.pref[a]};
        mid[a] = fw.ax[a].mid;
    }
    for (int64_t d0 = 0; d0 < n_dir; d0 += kFarChunk) {
        const int64_t nd = std::min(kFarChunk, n_dir - d0);
        // j tiles split until there are two waves per SIMD
        const int64_t waves = 3 * ((nd + 15) / 16);
        const int tiles = std::min(std::min(Kcp[0], Kcp[1]), Kcp[2]) / 16;
        args.jsplit = (int)std::max<int64_t>(1, std::min<int64_t>(tiles, (2048 + waves - 1) / waves));
        const int rows = 3 * args.jsplit;
        if (rows * nd > kFarPart) return hipErrorInvalidValue;
        hipLaunchKernelGGL(far_eval_kernel, dim3(blocks_of(nd, 16 * kFarWaves), rows), dim3(64 * kFarWaves), 0, stream,
                           dirs + d0, nd, args, s->far_part);
        hipLaunchKernelGGL(far_sum_kernel, dim3(blocks_of(nd)), dim3(256), 0, stream, dirs + d0, nd,
                           make_double3(mid[0], mid[1], mid[2]), s->far_part, rows, out + d0);
        const int per = (int)((nd + 16 * kWideGroups - 1) / (16 * kWideGroups)) * 16;
        hipLaunchKernelGGL(far_wide_kernel, dim3(blocks_of(nd, per)), dim3(64 * kWideWaves), 0, stream, dirs + d0, nd, per,
                           fw, scratch, out + d0);
    }
    return hipGetLastError();
}

hipError_t project_points(ProjectState** pst, const pstd_problem& p, const double dxb[3], double2* const acc[3],
                          const int64_t points[3], PhasorScale scale, const double3* obs, int64_t n_obs, double2* out,
                          hipStream_t stream, std::string* msg) {
    TRY(prepare(pst, p, acc, points, scale, stream));
    ProjectState* s = *pst;
    // the cell formula holds outside the box only
    unsigned flags = 0;
    TRY(check_points(s, p, dxb, obs, n_obs, &flags, stream));
    if (flags & 1) {
        *msg = "observation point inside the box or not finite";
        return hipErrorInvalidValue;
    }
    TRY(near_tables(s, p, stream));
    // a far field can be captured from here on (without memory for it, not)
    if (far_tables(s, p, dxb, stream)) (void)hipGetLastError();
    for (int f = 0; f < 6; ++f) {
        const FaceGeo g = face_geo(p, dxb, f);
        const int Nb = p.n[g.b], Nc = p.n[g.c], L = g.L, M = g.M;
        const int64_t ncell = (int64_t)L * M, np = (int64_t)Nb * Nc;
        const double2* Tb = s->near_tab + s->near_off[g.b];
        const double2* Tc = s->near_tab + s->near_off[g.c];
        // scratch: W [fld][p][Nc][L], Qg [fld][p][q][M][L], Q [cell][2][low terms]
        const size_t nW = (size_t)2 * kTerms * Nc * L, nQg = (size_t)2 * kPairs * ncell, nQ = (size_t)2 * kLow * ncell;
        TRY(ensure(&s->work, &s->work_bytes, (nW + nQg + nQ) * sizeof(double2)));
        double2* dW = s->work;
        double2* dQg = dW + nW;
        double2* dQ = dQg + nQg;
        const int64_t sW = (int64_t)Nc * L;
        // W_p = P [Nc x Nb] * Tb_p^T [Nb x L]
        TRY(zgemm(Nc, L, Nb, ZOp{s->phasors + s->face_off[f], Nb, 0, np}, ZOp{Tb, Nb, (int64_t)L * Nb, 0}, dW, L, sW,
                  kTerms * sW, kTerms, 2, ZOpts{false, false, true, false}, stream));
        // Q_pq = Tc_q [M x Nc] * W_p [Nc x L]
        TRY(zgemm(M, L, Nc, ZOp{Tc, Nc, (int64_t)M * Nc, 0}, ZOp{dW, L, 0, sW}, dQg, L, ncell, kTerms * ncell, kTerms,
                  2 * kTerms, {}, stream));
        hipLaunchKernelGGL(economise_kernel, dim3(blocks_of(ncell * kLow * 2)), dim3(256), 0, stream, dQg, ncell,
                           s->econ, 0.5 * g.db, 0.5 * g.dc, dQ);
        const int64_t bx = (n_obs + kNearThreads * kNearPoints - 1) / (kNearThreads * kNearPoints);
        const int splits = split_count(bx * (kNearThreads / 64), (ncell + kCellChunk - 1) / kCellChunk);
        const int64_t per = (ncell + splits - 1) / splits;
        TRY(ensure(&s->part, &s->part_bytes, (size_t)splits * n_obs * sizeof(double2)));
        auto near = (flags & 2) ? near_kernel<kNearPoints, false> : near_kernel<kNearPoints, true>;
        hipLaunchKernelGGL(near, dim3((unsigned)bx, (unsigned)splits), dim3(kNearThreads), 0, stream, obs, n_obs, p.k0,
                           g, dQ, per, s->part);
        hipLaunchKernelGGL(add_splits_kernel, dim3(blocks_of(n_obs)), dim3(256), 0, stream, s->part, splits, n_obs,
                           f > 0, out);
        // the next face reuses the scratch after these kernels, in stream order
    }
    return hipGetLastError();
}

hipError_t project_adjoint(ProjectState** pst, const pstd_problem& p, const double dxb[3], double2* const acc[3],
                           const int64_t points[3], double scale, const double3* obs, int64_t n_obs, const double2* g,
                           float2* inj, hipStream_t stream, std::string* msg) {
    // the state (tables, offsets) is shared with the forward projection
    TRY(prepare(pst, p, acc, points, real_scale(1.0), stream));
    ProjectState* s = *pst;
    unsigned flags = 0;
    TRY(check_points(s, p, dxb, obs, n_obs, &flags, stream));
    TRY(near_tables(s, p, stream));
    for (int f = 0; f < 6; ++f) {
        const FaceGeo geo = face_geo(p, dxb, f);
        const int Nb = p.n[geo.b], Nc = p.n[geo.c], L = geo.L, M = geo.M;
        const int64_t ncell = (int64_t)L * M, np = (int64_t)Nb * Nc;
        const double2* Tb = s->near_tab + s->near_off[geo.b];
        const double2* Tc = s->near_tab + s->near_off[geo.c];
        // scratch: low [fld][k][cell], Qbar [fld][p][q][cell], W [fld][Nc][9 L], F [fld][p][plane]
        const size_t nl = (size_t)2 * kLow * ncell, nQ = (size_t)2 * kPairs * ncell, nW = (size_t)2 * Nc * kTerms * L,
                     nF = (size_t)2 * kTerms * np;
        TRY(ensure(&s->work, &s->work_bytes, (nl + nQ + nW + nF) * sizeof(double2)));
        double2* dl = s->work;
        double2* dQ = dl + nl;
        double2* dW = dQ + nQ;
        double2* dF = dW + nW;
        const int64_t bx = (ncell + 127) / 128;
        const int splits = split_count(bx * 2 * kAdjGroups,
                                       std::min<int64_t>((n_obs + kAdjObsChunk - 1) / kAdjObsChunk, 16));
        const int64_t per = (n_obs + splits - 1) / splits;
        double2* ldst = dl;
        if (splits > 1) {
            TRY(ensure(&s->low, &s->low_bytes, (size_t)splits * nl * sizeof(double2)));
            ldst = s->low;
        }
        auto near = (flags & 2) ? near_adjoint_kernel<false> : near_adjoint_kernel<true>;
        hipLaunchKernelGGL(near, dim3((unsigned)bx, (unsigned)splits, kAdjGroups), dim3(128), 0, stream, obs, g, n_obs,
                           p.k0, geo, per, ldst);
        if (splits > 1)
            hipLaunchKernelGGL(add_splits_kernel, dim3(blocks_of((int64_t)nl)), dim3(256), 0, stream, s->low, splits,
                               (int64_t)nl, false, dl);
        hipLaunchKernelGGL(economise_adjoint_kernel, dim3(blocks_of((int64_t)nQ)), dim3(256), 0, stream, dl, ncell,
                           s->econ, 0.5 * geo.db, 0.5 * geo.dc, dQ);
        // Wbar[fld][c'][p L + l] = sum_qm conj(Tc[q M + m][c']) Qbar[fld][p][q M + m][l]
        TRY(zgemm(Nc, L, kTerms * M, ZOp{Tc, Nc}, ZOp{dQ, L, kTerms * ncell, kPairs * ncell}, dW, (int64_t)kTerms * L, L,
                  (int64_t)Nc * kTerms * L, kTerms, 2, ZOpts{true, true, false, false}, stream));
        // plane adjoint, one plane per p: Wbar_p [Nc x L] * conj(Tb_p) [L x Nb]
        TRY(zgemm(Nc, Nb, L, ZOp{dW, (int64_t)kTerms * L, L, (int64_t)Nc * kTerms * L}, ZOp{Tb, Nb, (int64_t)L * Nb, 0},
                  dF, Nb, np, kTerms * np, kTerms, 2, ZOpts{false, false, false, true}, stream));
        for (int fld = 0; fld < 2; ++fld)
            hipLaunchKernelGGL(conj_scale_kernel, dim3(blocks_of(np)), dim3(256), 0, stream, dF + fld * kTerms * np, np,
                               scale, inj + s->face_off[f] + fld * np);
        // the next face reuses the scratch after these kernels, in stream order
    }
    return hipGetLastError();
}

void project_free(ProjectState* s) {
    if (!s) return;
    void* ptrs[] = {s->phasors, s->work, s->part, s->low, s->flags, s->near_tab, s->econ, s->far_tab};
    for (void* q : ptrs) (void)hipFree(q);
    delete s;
}

}  // namespace pstd
