// xz_plane.h -- the z and x work between two fused y passes in one kernel, for grids
// whose (x, z) plane of one component fits in LDS: one workgroup per component and y.
//
// The fused y pass of one step leaves the half spectrum transformed along x and z only;
// the z inverse, x inverse, next x forward and next z forward that lead to the fused pass
// after it touch one (kx, z) plane at a time, so a workgroup can run all four on a plane
// held in LDS: one read and one write of the state where the separate passes make three,
// and one launch instead of three.  The butterflies, tables and rounding are those of the
// separate passes, so the results are the same bits.
//
// Measured (one pass replacing z inverse + x inverse-forward + z forward, us): 32^3 FP64
// 18 -> 9, 64^3 FP64 39 -> 15, 128^3 FP64 115 -> 51 (201 MB read and written: 3.9 TB/s,
// against 6-7 for a copy of that size in the last-level cache), 96^3 FP32 39 -> 25.  What
// bounds it: on small grids the latency of one load, two barriers and one store; on
// 128^3 the LDS (about 15 movements of the plane, 24 us of the 51, a third of it bank
// conflicts) and the vector ALU (16 us) beside 29 us of memory time, which the two waves
// per SIMD of the one workgroup a CU holds overlap only partly; in FP32 the vector ALU.
#pragma once
#include "passes.h"

namespace eifp {

template <typename T, class PZ, class PX>
struct XzCfg {
    static constexpr int M = PX::N, N = PZ::N;
    static constexpr int CW = 64 / PZ::T, GZ = (M + CW - 1) / CW;  // columns per wave, column groups
    static constexpr int RW = 64 / PX::T, GX = (N + RW - 1) / RW;  // rows per wave, row groups
    static constexpr int G = GZ > GX ? GZ : GX;
    static constexpr int LOOPS = (G + 15) / 16;
    static constexpr int W = (G + LOOPS - 1) / LOOPS, NT = 64 * W;
    // Rows of the plane in LDS have one empty element after every 16 and a pitch of 4 mod 16
    // elements: the stores of a radix-16 stage and the reads of four adjacent rows or
    // columns then fall in different banks (128^3 step 105.5 us FP64, 68.3 FP32 against
    // 109.7 and 71.2 with plain rows of odd pitch).  Planes that fit a CU only without the gaps
    // (FP64 96 x 96 and 16 x 512, for example) keep plain rows.  In FP32, where XzPair takes
    // planes of half a CU, the gaps shut six pairs out that would fit with plain rows (M x Nz 8,
    // 12 and 16 x 512, 48 x 192, 96 x 96, 192 x 48): those run the separate passes, and plain
    // rows have not been timed for them.
    static constexpr int padded() {
        int q = M - 1 + ((M - 1) >> 4) + 1;
        while (q % 16 != 4) ++q;
        return q;
    }
    static constexpr int bytes(int pitch) {
        return (N * pitch + (N + 2 * M) * TwParts<T>::value) * (int)sizeof(cpx<T>);
    }
    static constexpr int FULL = 160 * 1024, HALF = FULL / 2;
    static constexpr bool GAPS = bytes(padded()) <= FULL;
    static constexpr int PITCH = GAPS ? padded() : (M | 1), lds_bytes = bytes(PITCH);
    static __host__ __device__ constexpr int at(int k) { return GAPS ? k + (k >> 4) : k; }
    static constexpr bool PERSIST = lds_bytes > HALF;
};

// Views of the plane: a column (fixed kx, positions along z) and a row (fixed z).  Both
// stay within one wave, so their exchanges need only wave-scope ordering.
template <typename T, int PITCH>
struct PlaneCol {
    cpx<T>* p;  // plane + column offset
    bool active;
    __device__ __forceinline__ void st(int pos, cpx<T> a) {
        if (active) p[pos * PITCH] = a;
    }
    __device__ __forceinline__ cpx<T> ld(int pos) const { return p[pos * PITCH]; }
    __device__ __forceinline__ void sync() { wave_lds_sync(); }
    __device__ __forceinline__ void after_load() { wave_lds_sync(); }
};
template <typename T, class C>
struct PlaneRow {
    cpx<T>* p;  // plane + row offset
    bool active;
    __device__ __forceinline__ void st(int pos, cpx<T> a) {
        if (active) p[C::at(pos)] = a;
    }
    __device__ __forceinline__ cpx<T> ld(int pos) const { return p[C::at(pos)]; }
    __device__ __forceinline__ void sync() { wave_lds_sync(); }
    __device__ __forceinline__ void after_load() { wave_lds_sync(); }
};

// Grid: (G (+1: the finalize), 1, members): G workgroups share the member's 6 Ny planes.
// A workgroup that takes a whole CU (PERSIST) runs several planes, loading the next one's
// first group under the current one's x phase (128^3 FP64: pass 65 -> 53 us); the finalize is then workgroup 0's, since
// one workgroup more than the CUs hold would run alone at the end.
// X_FWD reads state and writes work, X_INV reads work and writes state, X_INVFWD runs in
// place on work.
template <typename T, class PZ, class PX, int KIND>
__global__ void __launch_bounds__((XzCfg<T, PZ, PX>::NT))
k_xz(const MemberDesc<T>* __restrict__ md, int ny, long cs, const cpx<T>* __restrict__ twz,
     const cpx<T>* __restrict__ twx, int fin_nparts) {
    using C = XzCfg<T, PZ, PX>;
    constexpr int M = C::M, N = C::N, PITCH = C::PITCH, EZ = PZ::E, EX = PX::E, TZ = PZ::T, TX = PX::T;
    static_assert(N * PITCH * (int)sizeof(cpx<T>) >= C::W * 2 * INV_NPART * (int)sizeof(double), "finalize scratch");
    __shared__ cpx<T> s_p[N * PITCH];
    __shared__ cpx<T> s_tz[N * TwParts<T>::value];
    __shared__ cpx<T> s_tx[2 * M * TwParts<T>::value];
    const MemberDesc<T>& mem = md[blockIdx.z];
    const int nwg = (int)gridDim.x - (!C::PERSIST && fin_nparts > 0 ? 1 : 0), nplanes = 6 * ny;
    if (!C::PERSIST && (int)blockIdx.x >= nwg) {  // the finalize (uniform per workgroup)
        finalize_member<INV_NPART, C::NT>(mem.partials, fin_nparts, mem.inv, reinterpret_cast<double*>(s_p));
        return;
    }
    const int wave = (int)threadIdx.x >> 6, lane = (int)threadIdx.x & 63;
    const cpx<T>* src = KIND == X_FWD ? mem.state : mem.work;
    cpx<T>* dst = KIND == X_INV ? mem.state : mem.work;
    const long zstride = (long)ny * M;
    // z phase: lane (c, t) of a wave holds positions t + TZ m of column c of its group
    const int zc = lane % C::CW, zt = lane / C::CW;
    const unsigned cbytes = (unsigned)cs * sizeof(cpx<T>);
    const unsigned sstep = (unsigned)(TZ * zstride) * sizeof(cpx<T>);
    auto col_of = [&](int g, bool& active) {
        const int col = g * C::CW + zc;
        active = M % C::CW == 0 || col < M;
        return active ? col : M - 1;
    };
    // plane p: component p / Ny, y = p % Ny
    auto voff_of = [&](int y, int col) { return (unsigned)(zt * zstride + (long)y * M + col) * sizeof(cpx<T>); };
    // x phase: lane (t, r) holds positions t + TX m of row r of its group
    const int xt = lane % TX, xr = lane / TX;
    auto row_of = [&](int g, bool& active) {
        const int z = g * C::RW + xr;
        active = N % C::RW == 0 || z < N;
        return active ? z : N - 1;
    };
    bool active;
    int p = (int)blockIdx.x;
    int comp = p / ny, y = p - comp * ny;
    cpx<T> nv[KIND == X_FWD ? EX : EZ];  // the plane's first group
    auto load_first = [&](int comp_, int y_) {
        bool a;
        if constexpr (KIND == X_FWD) {
            const cpx<T>* in = src + comp_ * cs + ((long)row_of(wave < C::GX ? wave : 0, a) * ny + y_) * M;
#pragma unroll
            for (int i = 0; i < EX; ++i) nv[i] = in[xt + TX * m_first<PX>(i)];
        } else {
            load_col<T, PZ>(nv, make_rsrc(src + comp_ * cs, cbytes), voff_of(y_, col_of(wave < C::GZ ? wave : 0, a)), sstep);
        }
    };
    load_first(comp, y);
    if (C::PERSIST && fin_nparts > 0 && blockIdx.x == 0) {
        finalize_member<INV_NPART, C::NT>(mem.partials, fin_nparts, mem.inv, reinterpret_cast<double*>(s_p));
        // (the barrier below comes before the plane is written)
    }
    stage_table_plan<PZ>(s_tz, twz);
    stage_table(s_tx, twx, 2 * M);
    __syncthreads();
    while (p < nplanes) {  // uniform over the workgroup
        const int pn = p + nwg, compn = pn / ny, yn = pn - compn * ny;
        if constexpr (KIND != X_FWD) {
            cpx<T> v[EZ];
            const __amdgpu_buffer_rsrc_t r = make_rsrc(src + comp * cs, cbytes);
            for (int g = wave; g < C::GZ; g += C::W) {
                const int col = col_of(g, active);
                if (C::GZ <= C::W || g == wave) {
#pragma unroll
                    for (int i = 0; i < EZ; ++i) v[i] = nv[i];
                } else {
                    load_col<T, PZ>(v, r, voff_of(y, col), sstep);
                }
                PlaneCol<T, PITCH> lds{s_p + C::at(col), active};
                fft_pencil<PZ, true, kStagedTw>(v, zt, lds, s_tz);
                lds.after_load();
#pragma unroll
                for (int i = 0; i < EZ; ++i) lds.st(zt + TZ * m_last<PZ>(i), v[i]);
            }
            __syncthreads();
            if (C::PERSIST && pn < nplanes) load_first(compn, yn);
        }
        {
            cpx<T> v[EX];
            for (int g = wave; g < C::GX; g += C::W) {
                const int z = row_of(g, active);
                PlaneRow<T, C> lds{s_p + z * PITCH, active};
                const long grow = ((long)z * ny + y) * M;
                if constexpr (KIND == X_FWD) {
                    if (C::GX <= C::W || g == wave) {
#pragma unroll
                        for (int i = 0; i < EX; ++i) v[i] = nv[i];
                    } else {
#pragma unroll
                        for (int i = 0; i < EX; ++i) v[i] = src[comp * cs + grow + xt + TX * m_first<PX>(i)];
                    }
                } else {
#pragma unroll
                    for (int i = 0; i < EX; ++i) v[i] = lds.ld(xt + TX * m_first<PX>(i));
                    x_inverse_row<T, PX, true>(v, xt, lds, s_tx);
                }
                if constexpr (KIND == X_INV) {
                    store_row<T, PX, true>(dst + comp * cs + grow, v, xt, active);
                } else {
                    if constexpr (KIND == X_INVFWD) {
                        // the physical row as materialised values (see x_invfwd_body)
#pragma unroll
                        for (int i = 0; i < EX; ++i) asm volatile("" : "+v"(v[i].x), "+v"(v[i].y));
                        last_to_first<PX>(v);
                        lds.after_load();  // the inverse's last exchange read
                    }
                    x_forward_row<T, PX>(v, xt, lds, s_tx);
                    lds.after_load();  // the split's partners read
#pragma unroll
                    for (int i = 0; i < EX; ++i) lds.st(xt + TX * m_last<PX>(i), v[i]);
                }
            }
        }
        __syncthreads();
        if constexpr (KIND != X_INV) {
            if (KIND == X_FWD && C::PERSIST && pn < nplanes) load_first(compn, yn);
            const __amdgpu_buffer_rsrc_t r = make_rsrc(dst + comp * cs, cbytes);
            for (int g = wave; g < C::GZ; g += C::W) {
                const int col = col_of(g, active);
                PlaneCol<T, PITCH> lds{s_p + C::at(col), active};
                cpx<T> v[EZ];
#pragma unroll
                for (int i = 0; i < EZ; ++i) v[i] = lds.ld(zt + TZ * m_first<PZ>(i));
                lds.after_load();
                fft_pencil<PZ, false, kStagedTw>(v, zt, lds, s_tz);
                store_col<T, PZ>(v, r, voff_of(y, col), sstep, active);
            }
            // the next plane's z inverse writes the columns this wave has read; its x
            // forward writes rows
            if (KIND == X_FWD && C::PERSIST) __syncthreads();
        }
        if (!C::PERSIST) break;
        p = pn;
        comp = compn;
        y = yn;
    }
}

}  // namespace eifp
