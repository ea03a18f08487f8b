// FDTD variant of the step (Section 2.2.1; its bound Section 2.3.1): the eighth-order central stencil of
// Eq. y_stencil (coefficients of Eq. stencil_alpha) along every axis, the
// central-difference update of Eq. FDTDupdatePsi with the potential, the
// wall consistency terms of Eqs. FDTDpsi_extraJminus1-FDTDpsiJplus4 and the
// mask of Eq. expmask, in one kernel per step.
//
// The wall terms of a cell c sum, over the axes a and the stencil offsets
// l, alpha_l [T(c) - T(c +- l e_a)] psi_inc(c +- l e_a), T = 1 on the
// total-field box.  With the separable incident wave this is
// sum_a D_a(i_a) prod_{b != a} Z_b(i_b) times the step's time factor, with
// the 1D tables Z_b = T_b e^{i kh_b x_b} and D_a = -C_a e^{i kh_a x_a} /
// dxb_a^2, C_a(i) = sum_l alpha_l sum_pm [T_a(i) - T_a(i pm l)]
// e^{pm i kh_a l dxb_a}: the same form as the taper source of the spectral
// scheme, so the same per-axis tables carry it.
//
// A workgroup owns a 32 x kFY tile of (x, y) columns and a run of z planes.
// Each thread keeps the nine values psi(z-4 .. z+4) of its column in VGPRs
// (the z stencil) and the plane z of the tile with a 4-cell halo is staged
// in LDS (the x and y stencils), in two buffers so that one barrier per plane
// is enough.  The loads of plane z + 2 (the halo cells, the next column value,
// psi^{n-1} and V) are issued right after plane z is staged, so they are in
// flight while planes z and z + 1 are computed; the z factors come from LDS,
// because a load of them from memory would return behind all of those.
// The grid is periodic (indices wrap), like the spectral passes.
#include "dft.hpp"
#include "internal.hpp"

namespace pstd {

namespace {

constexpr int kFX = 32;   // tile x (one wave row)
constexpr int kFH = 4;    // stencil reach
constexpr int kCUs = 256;
constexpr int kFZ = 16;   // z planes per workgroup at most
constexpr int kSX = kFX + 2 * kFH;

__device__ __forceinline__ int wrap(int i, int n) {
    i %= n;
    return i < 0 ? i + n : i;
}

typedef float float2_vec __attribute__((ext_vector_type(2)));

// Bound by the arithmetic and the LDS reads of a plane in turn with its
// barrier: about 90 vector and 57 scalar instructions and 21 LDS accesses per
// wave and plane, with psi 8 B read 1.5 times (runs overlap by eight planes)
// and 20 B of other traffic per cell next to it (160^3: 18 us of copy time).
// Everything that a plane loads has a register set of its own, three deep, so
// that no copy of a value just loaded waits for it.  16 planes unrolled: the
// column rotates by names instead of moves.  160^3: 27.2 -> 23.5 us, 288^3
// 181 -> 146 us, 98 x 134 x 150 23.6 -> 17.0, 48 x 64 x 80 16.1 -> 6.9.
// NTL: psi^{n-1}, read here for the last time, comes in with non-temporal
// loads (chosen for fields beyond the Infinity Cache, which then keeps the
// psi^{n+1} this step writes for the next).
template <bool NTL, int kFY>
__global__ __launch_bounds__(kFX * kFY) __attribute__((amdgpu_waves_per_eu(4))) void fdtd_kernel(FdtdArgs a, int run,
                                                                                                  int koff) {
    constexpr int kSY = kFY + 2 * kFH;
    __shared__ float2 s[2][kSY * (kSX + 1) + 32];
    __shared__ float2 s_zt[kFZ], s_dz[kFZ];
    __shared__ float s_gam[kFZ];
    const int tx = threadIdx.x, ty = threadIdx.y;
    const int t = ty * kFX + tx;
    const int nx = a.nx, ny = a.ny, nz = a.nz;
    const int64_t nstep = a.ctr[0] + koff;
    if (nstep >= a.ctr[1]) return;  // whole workgroup, before any barrier
    const float2* __restrict__ psi = (nstep & 1) ? a.buf[1] : a.buf[0];
    float2* __restrict__ old = (nstep & 1) ? a.buf[0] : a.buf[1];
    // Workgroups are dealt round-robin to the 8 XCDs (blockIdx mod 8); give
    // each XCD a contiguous run of tiles (x fastest, then y, then z) instead,
    // so that the halo rows and planes a tile shares with its neighbours meet
    // in one L2.  A bijection of [0, G).
    const int gx = (nx + kFX - 1) / kFX, gy = (ny + kFY - 1) / kFY;
    const int G = (int)gridDim.x, gb = (int)blockIdx.x, xcd = gb & 7;
    const int gt = xcd * (G >> 3) + min(xcd, G & 7) + (gb >> 3);
    const int bx = (gt % gx) * kFX, by = ((gt / gx) % gy) * kFY;
    const int bz = gt / (gx * gy);
    const int x = bx + tx, y = by + ty;
    const bool valid = x < nx && y < ny;
    const int xw = wrap(x, nx), yw = wrap(y, ny);
    // a plane holds fewer than 2^31 cells
    const int col = xw + nx * yw;
    const int64_t plane = (int64_t)nx * ny;
    const int z0 = bz * run;
    const int z1 = min(z0 + run, nz);

    if (t < z1 - z0) {
        s_zt[t] = a.zt[2][z0 + t];
        s_dz[t] = a.dz[2][z0 + t];
        s_gam[t] = a.gam[2][z0 + t];
    }
    // the column psi(z0-4 .. z0+5); at plane z, q[(r + z - z0) mod Q] holds
    // psi(z - 4 + r)
    constexpr int Q = 2 * kFH + 3;
    float2 q[Q];
    unroll<Q - 1>([&](auto i) {
        constexpr int r = decltype(i)::value;
        q[r] = (psi + plane * wrap(z0 - kFH + r, nz))[col];
    });
    // per-column factors of the mask and of the wall terms
    const float2 Zx = a.zt[0][xw], Dx = a.dz[0][xw];
    const float2 Zy = a.zt[1][yw], Dy = a.dz[1][yw];
    const float2 SA = cadd(cmul(Dx, Zy), cmul(Zx, Dy));
    const float2 SB = cmul(Zx, Zy);
    const float gxy = a.gam[0][xw] * a.gam[1][yw];
    const float2 sigma = a.sigma_tab[nstep];

    // this thread's halo cells of the staged tile (no corners), fixed for the
    // run: LDS slot and column offset
    constexpr int kHaloY = 2 * kFH * kFX, kHalo = kHaloY + 2 * kFH * kFY;
    constexpr int kSlots = (kHalo + kFX * kFY - 1) / (kFX * kFY);
    int hslot[kSlots];
    int hcol[kSlots];
    unroll<kSlots>([&](auto i) {
        constexpr int j = decltype(i)::value;
        const int e = t + j * kFX * kFY;
        int r, c;
        if (e < kHaloY) {
            r = e / kFX, c = kFH + e % kFX;
            if (r >= kFH) r += kFY;
        } else {
            r = kFH + (e - kHaloY) / (2 * kFH), c = (e - kHaloY) % (2 * kFH);
            if (c >= kFH) c += kFX;
        }
        hslot[j] = e < kHalo ? r * (kSX + 1) + c : kSY * (kSX + 1) + (t & 31);  // of the padded rows; past the tile for none
        hcol[j] = e < kHalo ? wrap(bx + c - kFH, nx) + nx * wrap(by + r - kFH, ny) : 0;
    });
    // loads of plane z, issued two planes ahead: the halo cells and the
    // epilogue operands psi^{n-1} and V of its cell.  Past the run (mask 0) the
    // first cell of the last plane stands in: a branch would cost waits.
    float2 hv[3][kSlots], po[3];
    float vv[3];
    auto load_plane = [&](auto set, int z, int mask) {
        constexpr int b = decltype(set)::value;
        const float2* pz = psi + plane * z;
        unroll<kSlots>([&](auto i) {
            constexpr int j = decltype(i)::value;
            hv[b][j] = pz[hcol[j] & mask];
        });
        const int c = col & mask;
        if constexpr (NTL) {
            const float2_vec v = __builtin_nontemporal_load((const float2_vec*)(old + plane * z) + c);
            po[b] = make_float2(v.x, v.y);
        } else {
            po[b] = (old + plane * z)[c];
        }
        vv[b] = (a.v2 + plane * z)[c];
    };
    load_plane(std::integral_constant<int, 0>{}, z0, -1);
    load_plane(std::integral_constant<int, 1>{}, min(z0 + 1, z1 - 1), -1);

    int zn = wrap(z0 + kFH + 2, nz);
    unroll<kFZ>([&](auto i) {
        constexpr int o = decltype(i)::value;  // the plane's place in the run
        const int z = z0 + o;
        if (z >= z1) return;
        // stage plane z: the own column value and the prefetched halo
        float2* sp = s[o & 1] + (ty + kFH) * (kSX + 1) + tx + kFH;
        *sp = q[(o + kFH) % Q];
        unroll<kSlots>([&](auto i) {
            constexpr int j = decltype(i)::value;
            s[o & 1][hslot[j]] = hv[o % 3][j];
        });
        __syncthreads();
        load_plane(std::integral_constant<int, (o + 2) % 3>{}, min(z + 2, z1 - 1), z + 2 < z1 ? -1 : 0);
        q[(o + Q - 1) % Q] = (psi + plane * zn)[col];
        zn = zn + 1 == nz ? 0 : zn + 1;
        if (valid) {
            const float2 c0 = q[(o + kFH) % Q];
            float2 k = cscale(c0, a.kc);
            unroll<kFH>([&](auto i) {
                constexpr int l = decltype(i)::value + 1;
                k = cadd(k, cscale(cadd(sp[-l], sp[l]), a.k[0][l - 1]));
                k = cadd(k, cscale(cadd(sp[-l * (kSX + 1)], sp[l * (kSX + 1)]), a.k[1][l - 1]));
                k = cadd(k, cscale(cadd(q[(o + kFH - l) % Q], q[(o + kFH + l) % Q]), a.k[2][l - 1]));
            });
            const float2 src = cadd(cmul(SA, s_zt[o]), cmul(SB, s_dz[o]));
            const float2 qq = cadd(cadd(k, cscale(c0, vv[o % 3])), cmul(sigma, src));
            const float g = gxy * s_gam[o];
            // psi^{n+1} = Gamma (psi^{n-1} - i q)
            (old + plane * z)[col] = make_float2(g * (po[o % 3].x + qq.y), g * (po[o % 3].y - qq.x));
        }
    });
}

}  // namespace

const double kFdtdAlpha[5] = {-205.0 / 72.0, 8.0 / 5.0, -1.0 / 5.0, 8.0 / 315.0, -1.0 / 560.0};

hipError_t launch_fdtd(const FdtdArgs& a, int koff, hipStream_t stream) {
    // psi pair and V: 20 B per cell
    const bool ntl = 20.0 * (double)a.nx * a.ny * a.nz > kInfinityCacheBytes;
    const int gx = (a.nx + kFX - 1) / kFX, gy = (a.ny + 7) / 8;
    // Four workgroups of 256 threads per CU, in one round: shorter runs start
    // more workgroups on a small grid, longer ones load fewer planes twice.
    // 48 x 64 x 80: 12.7 us with runs of 16, 6.85 with 3, 8.6 with 1;
    // 98 x 134 x 150: 19.6 with 16, 17.0 with 10, 18.1 with 6; 160^3: 24.0
    // with 16, 26.0 with 10.
    const int run = (int)std::min<int64_t>(kFZ, std::max<int64_t>(3, ((int64_t)a.nz * gx * gy + 4 * kCUs - 1) / (4 * kCUs)));
    // Tiles of 16 rows load fewer halo cells; where the runs are long and no
    // row is padded for it (288^3: 145.9 against 149.7 us, 160^3: 23.5 against
    // 24.0; 98 x 134 x 150: 21.2 against 19.6)
    const bool tall = run == kFZ && gy % 2 == 0;
    const dim3 grid((unsigned)(gx * (tall ? gy / 2 : gy) * ((a.nz + run - 1) / run))), block(kFX, tall ? 16 : 8);
    if (ntl)
        hipLaunchKernelGGL((tall ? fdtd_kernel<true, 16> : fdtd_kernel<true, 8>), grid, block, 0, stream, a, run, koff);
    else
        hipLaunchKernelGGL((tall ? fdtd_kernel<false, 16> : fdtd_kernel<false, 8>), grid, block, 0, stream, a, run, koff);
    return hipGetLastError();
}

}  // namespace pstd
