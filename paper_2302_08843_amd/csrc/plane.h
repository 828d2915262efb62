// plane.h -- the y and z transforms with the spectral product in one kernel,
// for grids whose y-z plane of the three components fits a compute unit.
#pragma once
#include "passes.h"

namespace mmx {

// Value of lane ^ X (X = 1, 2: data-parallel primitives within a quad; 4: a
// swizzle).
template <int X>
__device__ __forceinline__ int lane_xor_bits(int v)
{
    if constexpr (X == 1)
        return __builtin_amdgcn_update_dpp(0, v, 0xB1, 0xF, 0xF, true);  // quad [1,0,3,2]
    else if constexpr (X == 2)
        return __builtin_amdgcn_update_dpp(0, v, 0x4E, 0xF, 0xF, true);  // quad [2,3,0,1]
    else
        return __builtin_amdgcn_ds_swizzle(v, (X << 10) | 0x1F);
}
template <int X>
__device__ __forceinline__ float lane_xor(float v)
{
    return __int_as_float(lane_xor_bits<X>(__float_as_int(v)));
}
template <int X>
__device__ __forceinline__ double lane_xor(double v)
{
    return __hiloint2double(lane_xor_bits<X>(__double2hiint(v)),
                            lane_xor_bits<X>(__double2loint(v)));
}

// Shape of the plane kernel.  The zero-padded y transform of length Py = 2 YP
// splits into two unpadded ones of length YP >= ny, for even (q = 0) and odd
// (q = 1) frequencies ky = 2 p + q of x[j] and x[j] exp(-2 pi i j / Py); their
// inverses add up.  EY: registers per thread of the y transforms.  LZ lanes
// hold one z pencil: lane r owns the frequencies kz = LZ k + r, k < RZ, of
// x[k] folded and modulated the same way (LZ = 1: the whole padded pencil).
// NQ = 2: both q at once in two halves of the block, NQ = 1: one after the
// other; NTQ threads per q.
template <typename T, int YP, int EY, int PZ, int LZ, int NQ, int NTQ>
struct PlaneG {
    using S = FFTShape<YP, EY>;
    static constexpr int kE = S::kE, kT = S::kT;
    static constexpr int kP2 = PZ > 1 ? PZ / 2 : 1;  // most layers
    static constexpr int kRZ = PZ / LZ;
    static constexpr int kF = LZ > 1 ? LZ / 2 : 1;
    static constexpr int kNTQ = NTQ, kNT = NTQ * NQ;
    static constexpr int kIZ = YP * LZ / NTQ;        // pencils per lane group
    static constexpr int kRows = 3 * kP2;            // (component, layer) rows
    // LDS rows of one q: block 0 exchanges the z spectrum of all lanes (LZ = 1)
    // or of the lanes of one parity through them
    static constexpr int kLR = LZ == 1 ? 3 * PZ : kRows;
    static constexpr int kRP = S::kLds;              // LDS pitch of a row
    static constexpr int kRPP = kNTQ / kT;           // rows transformed at a time
    static constexpr int kIT = (kRows + kRPP - 1) / kRPP;
    // kernel entries a lane loads ahead of its transforms, as registers allow
    static constexpr int kKC = kNT <= 512 ? (sizeof(T) == 4 ? 8 : 4) : (sizeof(T) == 4 ? 4 : 2);
    static constexpr long kBytes =
        ((long)NQ * kLR * kRP + 2 * YP + 2 * PZ) * (long)sizeof(cx<T>);
    static constexpr bool kOK = kT <= 64 && kNT <= 1024 && kIZ * NTQ == YP * LZ && NTQ % kT == 0 &&
                                NTQ % LZ == 0 && kBytes <= 160 * 1024 - 1024;
};

// Offset of component 0 at kzf = 0 of the frequencies of parity q inside one
// kx column of the spectral kernel's plane layout, [kx][q][6][Pz/2+1][n_q]
// with ky = 2 i + q, i < n_q: n_0 = YP/2 + 1, n_1 = YP/2.
__host__ __device__ inline long plane_koff(int q, int YP, int hz)
{
    return q ? 6L * hz * (YP / 2 + 1) : 0;
}
__host__ __device__ inline int plane_kn(int q, int YP) { return YP / 2 + (q ? 0 : 1); }

// F2 + F3 + I2 in one: a block owns the column kx of the x spectrum, in place,
// holds its three nz x ny planes in LDS and runs the y transforms (rows,
// wave-local), the z transforms with the product (a pencil per LZ lanes, in
// registers; the lanes of a pencil exchange by register moves only) and the
// inverses.  Neither the y nor the z padding is ever stored.  The spectrum is
// laid out for it, ST[kx][3][nz][nyp] with y fastest (nyp = ny rounded up to
// even), so that a block reads and writes one contiguous piece.  The columns
// kx = 0 and kx = M of a real transform are real: column 0 holds both as
// Z = X_0 + i X_M, and since their products are Hermitian too,
// H = (K_0 + K_M)/2 Z(k) + (K_0 - K_M)/2 conj Z(-k) returns h_0 + i h_M.  So
// M blocks cover M + 1 columns, and a grid of 129 to 256 cells along x takes
// exactly one block per compute unit.  A batch of requests takes M blocks
// each (spectra bstride apart).
//
// Against the three passes it replaces, the y-transformed spectrum (twice the
// size of the x one) is neither written nor read twice, and two launches go.
// A field evaluation takes, before and after (us): FP32 64x64x2 27.4 / 16.1,
// 128x128x2 32.3 / 19.3, 256x64x4 30.7 / 21.0, 256x256x8 60.4 / 48.3,
// 256x256x16 107 / 91, 512x256x16 190 / 167; FP64 32x32x4 25.1 / 18.0,
// 256x256x4 61.4 / 50.5, 256x256x8 92.3 / 80.1.  Single layers, whose z pass
// along y held 8 columns in one wavefront for 12 us at any small size: FP32
// 64x64x1 21.0 / 15.0, 512x512x1 52.9 / 31.6; FP64 19.8 / 16.5, 63.7 / 45.6.
// It is bound by VALU issue and by the latency of its phases (a plane of 104 KB
// leaves one block per compute unit, whose wavefronts meet at every barrier;
// VALUs busy about half of the time), not by memory.  Hence as many threads as fit 128 registers, where that
// takes few spills (256x256x8: 1024 threads 48.3, 512 threads 52.2; a version
// that spilled 50 registers took 100x500x3 from 41 to 65): all shapes fit but
// the two of 1024 threads in FP32 that run one q after the other, (256, 32)
// with 23 registers spilled, the one of 256x256x16 above, and (512, 16) with
// 47.  No branches inside the phases (layers beyond nz are rows of zeros), and
// a spectrum with y fastest (reading columns of the row-major one: 256x256x8
// 81).
template <typename T, int YP, int EY, int PZ, int LZ, int NQ, int NTQ>
__global__ __launch_bounds__((PlaneG<T, YP, EY, PZ, LZ, NQ, NTQ>::kNT)) void k_plane(
    cx<T>* __restrict__ ST, cx<T>* __restrict__ scratch, const T* __restrict__ KT, int ny, int nz,
    int nyp, int M, long nblocks, long bstride, const cx<T>* __restrict__ tw, int Lmax)
{
    using G = PlaneG<T, YP, EY, PZ, LZ, NQ, NTQ>;
    constexpr int kE = G::kE, kT = G::kT, RZ = G::kRZ, P2 = G::kP2, F = G::kF, IT = G::kIT;
    constexpr int RP = G::kRP, PY = 2 * YP, HZ = PZ / 2 + 1;
    __shared__ __attribute__((aligned(32))) cx<T> plane[NQ * G::kLR * RP];
    __shared__ cx<T> twy[PY];  // exp(-2 pi i n / Py)
    // per lane r of a pencil: forward exp(-2 pi i k r / Pz), and for the inverse
    // the same at its own order of the outputs (zinv below)
    __shared__ __attribute__((aligned(32))) cx<T> twf[LZ > 1 ? PZ : 1], twi[LZ > 1 ? PZ : 1];
    const long lb = xcd_logical();
    if (lb >= nblocks) return;
    const int kx = (int)(lb % M), nrows = 3 * nz;
    cx<T>* S = ST + (lb / M) * bstride + (long)kx * nrows * nyp;
    const bool packed = kx == 0;
    // the q of a wavefront is uniform unless two share one
    const int gv = (int)threadIdx.x / G::kNTQ, s = (int)threadIdx.x % G::kNTQ;
    const int g = G::kNTQ % 64 == 0 ? __builtin_amdgcn_readfirstlane(gv) : gv;
    int t = s % kT, rl = s / kT;  // y phase: thread t of row slot rl
    constexpr int IZ = G::kIZ, PS = G::kNTQ / LZ;
    int p0 = s / LZ, r = s % LZ;  // z phase: lane r of pencils p0 + PS iz

    // row c P2 + k of the plane is layer k of component c; layers beyond nz and
    // cells beyond ny read element 0 and count as zero
    auto load = [&](int it, cx<T> (&v)[kE]) {
        const int row = it * G::kRPP + rl, c = row / P2, k = row % P2;
        const bool rok = row < G::kRows && k < nz;
        const unsigned o = (unsigned)((c * nz + k) * nyp + t);
#pragma unroll
        for (int e = 0; e < kE; ++e) {
            const bool ok = rok && t + e * kT < ny;
            const cx<T> a = elem<true>(S, ok ? o + (unsigned)(e * kT) : 0u);
            v[e] = ok ? a : cx<T>{0, 0};
        }
    };
    cx<T> v0[kE];  // the first rows, in flight with the twiddles
    load(0, v0);
    for (int n = threadIdx.x; n < PY; n += G::kNT) twy[n] = tw[n * (Lmax / PY)];
    if constexpr (LZ > 1) {
        for (int n = threadIdx.x; n < PZ; n += G::kNT) {
            const int rr = n / RZ, k = n % RZ, ki = k ^ (rr >= F ? RZ / 2 : 0);
            twf[n] = tw[(k * rr) % PZ * (Lmax / PZ)];
            twi[n] = tw[((ki + RZ * (rr % F)) * rr) % PZ * (Lmax / PZ)];
        }
    }
    __syncthreads();

    cx<T>* pl = plane + (NQ == 2 ? g * G::kLR * RP : 0);
#pragma unroll
    for (int qs = 0; qs < 2 / NQ; ++qs) {
        // the odd half recomputes its addresses and reads its rows again: held
        // across the even half they would not fit the registers
        if (qs) asm volatile("" : "+v"(t), "+v"(rl), "+v"(p0), "+v"(r));
        const int q = NQ == 2 ? g : qs;
        // ---- y forward ----
#pragma unroll
        for (int it = 0; it < IT; ++it) {
            const int row = it * G::kRPP + rl;
            cx<T> v[kE];
            if (it == 0 && (NQ == 2 || qs == 0)) {
#pragma unroll
                for (int e = 0; e < kE; ++e) v[e] = v0[e];
            } else {
                load(it, v);
            }
            if (row < G::kRows) {
                cx<T>* L = pl + row * RP;
                if (q) {
#pragma unroll
                    for (int e = 0; e < kE; ++e) v[e] = cmul(v[e], twy[t + e * kT]);
                }
                WgFFT<T, YP, EY, -1, false, false, true>::run(v, t, L, 1, twy, 2);
                fft_sync<true>();  // the last exchange's reads precede these writes
#pragma unroll
                for (int i = 0; i < kE; ++i) L[G::S::out_index(t, i)] = v[i];
            }
        }
        __syncthreads();
        // ---- z forward, product, z inverse ----
        {
            // lane constants: w_LZ^(f r), and for the inverse w_LZ^((f ^ fr) - fr) r),
            // fr = r mod F
            cx<T> wf[F], wi[F];
            const int fr = r % F;
#pragma unroll
            for (int f = 1; f < F; ++f) {
                wf[f] = twy[((f * r) & (LZ - 1)) * (PY / LZ)];
                wi[f] = twy[((((f ^ fr) - fr) * r) & (LZ - 1)) * (PY / LZ)];
            }
            const T sb = r >= F ? (T)-1 : (T)1;  // (LZ > 1)
            auto fwd = [&](int p, cx<T> (&z)[3][RZ]) {
                cx<T> tz[RZ];
                if constexpr (LZ > 1) {
#pragma unroll
                    for (int k = 0; k < RZ; ++k) tz[k] = twf[r * RZ + k];
                }
#pragma unroll
                for (int c = 0; c < 3; ++c) {
                    const cx<T>* L = pl + c * P2 * RP + p;
                    if constexpr (LZ == 1) {
#pragma unroll
                        for (int k = 0; k < RZ; ++k) z[c][k] = k < P2 ? L[k * RP] : cx<T>{0, 0};
                        dft<RZ, -1, (RZ > 1)>(z[c]);
                    } else {
#pragma unroll
                        for (int k = 0; k < RZ; ++k) {
                            cx<T> a = L[k * RP];
#pragma unroll
                            for (int f = 1; f < F; ++f) a = cadd(a, cmul(L[(k + RZ * f) * RP], wf[f]));
                            z[c][k] = k ? cmul(a, tz[k]) : a;
                        }
                        dft<RZ, -1>(z[c]);
                    }
                    __builtin_amdgcn_sched_barrier(0);  // one component's loads at a time
                }
            };
            // The inverse: lane r adds to out[k + RZ f] its conj(w_Pz^((k + RZ f) r))
            // times the RZ-point inverse at k.  It keeps its values in the
            // order k ^ (RZ/2 for r >= F; from alternating the inputs' signs)
            // and f ^ fr, so that in each exchange it keeps the first half of
            // them and sends the second, and ends with the outputs
            // k0 + [0, RZ/2).  signs: whether the inputs' signs are still to
            // be alternated.
            const int k0 = LZ > 1 ? (r >= F ? RZ / 2 : 0) + RZ * fr : 0;
            auto inv = [&](int p, cx<T> (&z)[3][RZ], bool signs) {
                cx<T> tz[RZ];
                if constexpr (LZ > 1) {
#pragma unroll
                    for (int k = 0; k < RZ; ++k) tz[k] = twi[r * RZ + k];
                }
#pragma unroll
                for (int c = 0; c < 3; ++c) {
                    cx<T>* L = pl + c * P2 * RP + p;
                    if (LZ > 1 && signs) {
#pragma unroll
                        for (int k = 1; k < RZ; k += 2) z[c][k] = cscale(z[c][k], sb);
                    }
                    dft<RZ, 1>(z[c]);
                    if constexpr (LZ == 1) {
#pragma unroll
                        for (int k = 0; k < P2; ++k) L[k * RP] = z[c][k];
                    } else {
                        cx<T> o[P2];
#pragma unroll
                        for (int k = 0; k < RZ; ++k) {
                            o[k] = cmulc(z[c][k], tz[k]);
#pragma unroll
                            for (int f = 1; f < F; ++f) o[k + RZ * f] = cmulc(o[k], wi[f]);
                        }
                        auto add = [&](auto X, int n) {
                            constexpr int x = decltype(X)::value;
#pragma unroll
                            for (int i = 0; i < P2 / 2; ++i)
                                if (i < n)
                                    o[i] = {o[i].x + lane_xor<x>(o[i + n].x),
                                            o[i].y + lane_xor<x>(o[i + n].y)};
                        };
                        using X1 = std::integral_constant<int, 1>;
                        using X2 = std::integral_constant<int, 2>;
                        using X4 = std::integral_constant<int, 4>;
                        if constexpr (LZ == 2) {
                            add(X1{}, P2 / 2);
                        } else if constexpr (LZ == 4) {
                            add(X1{}, P2 / 2);
                            add(X2{}, P2 / 4);
                        } else {
                            add(X2{}, P2 / 2);
                            add(X1{}, P2 / 4);
                            add(X4{}, P2 / 8);
                        }
#pragma unroll
                        for (int i = 0; i < RZ / 2; ++i) L[(k0 + i) * RP] = o[i];
                    }
                    __builtin_amdgcn_sched_barrier(0);
                }
            };
            // entries (xx, yy, zz, xy, xz, yz) of the kernel column at o_col
            // and frequency (2 pp + q, kz)
            const int kn = plane_kn(q, YP);
            const unsigned kcol = 6u * HZ * (YP + 1);
            const unsigned kq = (unsigned)kx * kcol + (unsigned)plane_koff(q, YP, HZ);
            auto kload = [&](unsigned o_col, int pp, int kz, T (&m)[6]) {
                const bool my = 2 * pp + q > YP, mz = kz > PZ / 2;
                const int pf = my ? YP - q - pp : pp;
                const unsigned o = o_col + (unsigned)((mz ? PZ - kz : kz) * kn + pf);
#pragma unroll
                for (int e = 0; e < 6; ++e) m[e] = elem<true>(KT + e * HZ * kn, o);
            };
            // the signs of xy, xz, yz on the mirrored halves (odd: times sb)
            auto ksign = [&](int pp, int kz, T (&m)[6], bool odd) {
                const T sy = 2 * pp + q > YP ? (T)-1 : (T)1, sz = kz > PZ / 2 ? (T)-1 : (T)1;
                const T s0 = odd ? sb : (T)1;
                if (odd) {
                    m[0] *= s0;
                    m[1] *= s0;
                    m[2] *= s0;
                }
                m[3] *= s0 * sy;
                m[4] *= s0 * sz;
                m[5] *= s0 * sy * sz;
            };
            auto product = [](const T (&m)[6], const cx<T>& a, const cx<T>& b, const cx<T>& d,
                              cx<T> (&h)[3]) {
                h[0] = {m[0] * a.x + m[3] * b.x + m[4] * d.x, m[0] * a.y + m[3] * b.y + m[4] * d.y};
                h[1] = {m[3] * a.x + m[1] * b.x + m[5] * d.x, m[3] * a.y + m[1] * b.y + m[5] * d.y};
                h[2] = {m[4] * a.x + m[5] * b.x + m[2] * d.x, m[4] * a.y + m[5] * b.y + m[2] * d.y};
            };
            if (!packed) {
                constexpr int KC = cmin(RZ, G::kKC);  // kernel entries loaded ahead
#pragma unroll
                for (int iz = 0; iz < IZ; ++iz) {
                    const int p = p0 + PS * iz;
                    T m[KC][6];
#pragma unroll
                    for (int k = 0; k < KC; ++k) kload(kq, p, LZ * k + r, m[k]);
                    __builtin_amdgcn_sched_barrier(0);
                    cx<T> z[3][RZ];
                    fwd(p, z);
#pragma unroll
                    for (int kb = 0; kb < RZ; kb += KC) {
                        if (kb) {
#pragma unroll
                            for (int k = 0; k < KC; ++k) kload(kq, p, LZ * (kb + k) + r, m[k]);
                        }
#pragma unroll
                        for (int k = 0; k < KC; ++k) {
                            ksign(p, LZ * (kb + k) + r, m[k], LZ > 1 && (kb + k) % 2 == 1);
                            cx<T> h[3];
                            product(m[k], z[0][kb + k], z[1][kb + k], z[2][kb + k], h);
#pragma unroll
                            for (int c = 0; c < 3; ++c) z[c][kb + k] = h[c];
                        }
                        __builtin_amdgcn_sched_barrier(0);
                    }
                    inv(p, z, false);
                }
            } else {
                // block 0: the spectrum through LDS (lanes of even r, then of
                // odd r: kz and Pz - kz have one parity), both members of a
                // pair (k, -k) by one thread
                constexpr int NR = LZ == 1 ? 1 : 2, LP = LZ / NR, NS = RZ * LP;
                cx<T> z[IZ][3][RZ];
#pragma unroll
                for (int iz = 0; iz < IZ; ++iz) fwd(p0 + PS * iz, z[iz]);
#pragma unroll 1
                for (int rr = 0; rr < NR; ++rr) {
                    const bool mine = NR == 1 || (r & 1) == rr;
                    __syncthreads();  // the plane is read
                    if (mine) {
#pragma unroll
                        for (int i = 0; i < 3 * IZ * RZ; ++i)
                            pl[((i / RZ % 3 * RZ + i % RZ) * LP + r / NR) * YP + p0 +
                               PS * (i / (3 * RZ))] = z[i / (3 * RZ)][i / RZ % 3][i % RZ];
                    }
                    __syncthreads();
#pragma unroll 1
                    for (int i = s; i < NS * YP; i += G::kNTQ) {
                        // slot i / YP holds kz = NR * slot + rr
                        const int sl = i / YP, pp = i % YP, kz = NR * sl + rr;
                        const int kz2 = (PZ - kz) % PZ, p2 = (YP - q - pp) & (YP - 1);
                        const int i2 = (kz2 / NR) * YP + p2;
                        if (i2 < i) continue;
                        T m0[6], m1[6];
                        kload(kq, pp, kz, m0);
                        kload(kq + (unsigned)M * kcol, pp, kz, m1);
                        ksign(pp, kz, m0, false);
                        ksign(pp, kz, m1, false);
                        cx<T> a[3], b[3], u[3], w[3];
#pragma unroll
                        for (int e = 0; e < 6; ++e) {
                            const T ks = (T)0.5 * (m0[e] + m1[e]), kd = (T)0.5 * (m0[e] - m1[e]);
                            m0[e] = ks;
                            m1[e] = kd;
                        }
#pragma unroll
                        for (int c = 0; c < 3; ++c) {
                            a[c] = pl[c * NS * YP + i];
                            b[c] = cconj(pl[c * NS * YP + i2]);
                        }
                        product(m0, a[0], a[1], a[2], u);
                        product(m1, b[0], b[1], b[2], w);
#pragma unroll
                        for (int c = 0; c < 3; ++c) pl[c * NS * YP + i] = cadd(u[c], w[c]);
                        if (i2 != i) {
                            // at -k the entries xy and xz change sign
                            m0[3] = -m0[3];
                            m0[4] = -m0[4];
                            m1[3] = -m1[3];
                            m1[4] = -m1[4];
                            product(m0, b[0], b[1], b[2], u);
                            product(m1, a[0], a[1], a[2], w);
#pragma unroll
                            for (int c = 0; c < 3; ++c)
                                pl[c * NS * YP + i2] = {u[c].x + w[c].x, -(u[c].y + w[c].y)};
                        }
                    }
                    __syncthreads();
                    if (mine) {
#pragma unroll
                        for (int i = 0; i < 3 * IZ * RZ; ++i)
                            z[i / (3 * RZ)][i / RZ % 3][i % RZ] =
                                pl[((i / RZ % 3 * RZ + i % RZ) * LP + r / NR) * YP + p0 +
                                   PS * (i / (3 * RZ))];
                    }
                }
                __syncthreads();
#pragma unroll
                for (int iz = 0; iz < IZ; ++iz) inv(p0 + PS * iz, z[iz], true);
            }
        }
        __syncthreads();
        // ---- y inverse ----
#pragma unroll
        for (int it = 0; it < IT; ++it) {
            const int row = it * G::kRPP + rl;
            if (row < G::kRows) {
                cx<T>* L = pl + row * RP;
                cx<T> w[kE];
#pragma unroll
                for (int e = 0; e < kE; ++e) w[e] = L[t + e * kT];
                fft_sync<true>();  // these reads precede the first exchange
                WgFFT<T, YP, EY, 1, false, false, true>::run(w, t, L, 1, twy, 2);
                if (q) {
#pragma unroll
                    for (int i = 0; i < kE; ++i) w[i] = cmulc(w[i], twy[G::S::out_index(t, i)]);
                }
                fft_sync<true>();
#pragma unroll
                for (int i = 0; i < kE; ++i) L[G::S::out_index(t, i)] = w[i];
            }
        }
        __syncthreads();
        // out, two cells per thread: the sum of the two q (NQ = 1: the block's
        // share of the scratch spectrum holds the even one meanwhile)
        struct alignas(2 * sizeof(cx<T>)) cx2 {
            cx<T> a, b;
        };
        cx2* half = reinterpret_cast<cx2*>(scratch) + lb * ((long)nrows * nyp / 2);
        for (int i = threadIdx.x; i < G::kRows * (YP / 2); i += G::kNT) {
            const int row = i / (YP / 2), j = i % (YP / 2) * 2, c = row / P2, k = row % P2;
            if (k >= nz || j >= ny) continue;
            const unsigned o = (unsigned)((c * nz + k) * nyp + j) / 2;
            cx2 u = *reinterpret_cast<const cx2*>(plane + row * RP + j);
            if (NQ == 1 && q == 0) {
                elem<true>(half, o) = u;
                continue;
            }
            const cx2 w = NQ == 2 ? *reinterpret_cast<const cx2*>(plane + (G::kLR + row) * RP + j)
                                  : elem<true>(half, o);
            u.a = cadd(u.a, w.a);
            u.b = cadd(u.b, w.b);
            elem<true>(reinterpret_cast<cx2*>(S), o) = u;
        }
        if (NQ == 1) __syncthreads();  // the next q overwrites the plane
    }
}

// The shapes by padded y and z extents: MACRO(YP, EY, PZ, LZ, NQ, NTQ).
#define MMX_PLANE_F32(X)                                                                    \
    X(8, 4, 1, 1, 2, 8) X(8, 4, 4, 1, 2, 8) X(8, 4, 8, 2, 2, 16) X(8, 4, 16, 2, 2, 16)      \
    X(8, 4, 32, 4, 2, 32) X(8, 4, 64, 8, 2, 64) X(16, 4, 1, 1, 2, 16)                       \
    X(16, 4, 4, 1, 2, 16) X(16, 4, 8, 2, 2, 32) X(16, 4, 16, 2, 2, 32)                      \
    X(16, 4, 32, 4, 2, 64) X(16, 4, 64, 8, 2, 128) X(32, 8, 1, 1, 2, 32)                    \
    X(32, 8, 4, 1, 2, 32) X(32, 8, 8, 2, 2, 64) X(32, 8, 16, 2, 2, 64)                      \
    X(32, 8, 32, 4, 2, 128) X(32, 8, 64, 8, 2, 256) X(64, 8, 1, 1, 2, 64)                   \
    X(64, 8, 4, 1, 2, 64) X(64, 8, 8, 2, 2, 128) X(64, 8, 16, 2, 2, 128)                    \
    X(64, 8, 32, 4, 2, 256) X(128, 8, 1, 1, 2, 64) X(128, 16, 4, 1, 2, 128)                 \
    X(128, 16, 8, 2, 2, 256) X(128, 16, 16, 2, 2, 256) X(128, 16, 32, 4, 2, 512)            \
    X(256, 16, 1, 1, 2, 64) X(256, 16, 4, 1, 2, 256) X(256, 16, 8, 2, 2, 256)               \
    X(256, 16, 16, 2, 2, 512) X(256, 16, 32, 4, 1, 1024) X(512, 16, 1, 1, 2, 128)           \
    X(512, 16, 4, 1, 2, 512) X(512, 16, 8, 2, 2, 256) X(512, 8, 16, 2, 1, 1024)
#define MMX_PLANE_F64(X)                                                                    \
    X(8, 4, 1, 1, 2, 8) X(8, 4, 4, 1, 2, 8) X(8, 4, 8, 2, 2, 16) X(8, 4, 16, 4, 2, 32)      \
    X(8, 4, 32, 8, 2, 64) X(16, 4, 1, 1, 2, 16) X(16, 4, 4, 1, 2, 16)                       \
    X(16, 4, 8, 2, 2, 32) X(16, 4, 16, 4, 2, 64) X(16, 4, 32, 8, 2, 128)                    \
    X(32, 8, 1, 1, 2, 32) X(32, 8, 4, 1, 2, 32) X(32, 8, 8, 2, 2, 64)                       \
    X(32, 8, 16, 2, 2, 64) X(32, 8, 32, 4, 2, 128) X(64, 8, 1, 1, 2, 64)                    \
    X(64, 8, 4, 1, 2, 64) X(64, 8, 8, 2, 2, 128) X(64, 8, 16, 2, 2, 128)                    \
    X(64, 8, 32, 4, 2, 256) X(128, 8, 1, 1, 2, 64) X(128, 8, 4, 1, 2, 128)                  \
    X(128, 8, 8, 2, 2, 128) X(128, 8, 16, 2, 2, 256) X(128, 8, 32, 4, 1, 512)               \
    X(256, 8, 1, 1, 2, 128) X(256, 8, 4, 1, 2, 256) X(256, 8, 8, 2, 2, 256)                 \
    X(256, 8, 16, 2, 1, 512) X(512, 8, 1, 1, 2, 256) X(512, 8, 4, 1, 1, 512)                \
    X(512, 8, 8, 2, 1, 512)

template <typename T>
hipError_t launch_plane(const Plan& p);
template <>
hipError_t launch_plane<float>(const Plan& p);
template <>
hipError_t launch_plane<double>(const Plan& p);

#define MMX_PLANE_CASE(YP, EY, PZ, LZ, NQ, NTQ)                                              \
    if (p.P[1] == 2 * YP && p.P[2] == PZ) {                                                  \
        using V = cx<MMX_PLANE_T>;                                                           \
        using G = PlaneG<MMX_PLANE_T, YP, EY, PZ, LZ, NQ, NTQ>;                              \
        static_assert(G::kOK, "plane shape");                                                \
        k_plane<MMX_PLANE_T, YP, EY, PZ, LZ, NQ, NTQ>                                        \
            <<<xcd_grid(nb), G::kNT, 0, p.stream>>>(                                         \
                (V*)p.S2, (V*)p.S1, (const MMX_PLANE_T*)p.Khat, p.n[1], p.n[2],              \
                plane_pitch(p.n[1]), M, nb, plane_stride(p), (const V*)p.tw, p.Lmax);                  \
        return hipGetLastError();                                                            \
    }

}  // namespace mmx
