// fused_wide.h -- the fused y pass with one component per wave.
//
// A tile of B adjacent x columns of all six components is held in LDS.  Each wave
// transforms columns of one component (E values a lane), writes the spectrum to the tile,
// and after a barrier every thread propagates and sums modes of all six components from
// the tile; after another barrier the waves transform their component back and store it.
// A pencil lies in one wave, so its exchanges need no barrier, and a thread holds one
// component's values instead of six (k_fused) or three (k_fused_split): on small grids a
// tile's six waves fill the device where the other forms' one to four cannot, and in FP64
// at lengths 96 to 256 the freed registers hold 12 or 16 values a lane (fewer stages) and
// the next tile's loads.  The modes ky and -ky of a column are one thread's, which forms
// the phase and the coefficients once for both (a tenth of the pass's vector instructions).
//
// Measured (us, the form replaced / this one): 32^3 FP64 17 / 10, 64^3 FP64 24 / 14 and
// FP32 19 / 11, 128^3 FP64 54 / 42 (4.8 TB/s), 192^3 FP64 248 / 178 (3.8 TB/s), 256^3 FP64
// 419 / 376 (4.3 TB/s).  Bound by
// the latency of a load, two barriers and a store on small grids; above, a CU holds one
// workgroup, whose memory, LDS and arithmetic phases (192^3: 123, 61 and 44 us of the
// 178) only the loads of the next tile overlap.
#pragma once
#include "kernels.h"

namespace eifp {

template <typename T, class P>
struct WideCfg {
    static constexpr int N = P::N, CW = 64 / P::T, B = CW;
    // Waves of a workgroup: six, one per component; in FP32 at 128 and 256, whose two
    // workgroups a CU keep the vector ALU busy, eight, so that they load the four SIMDs alike
    // and take a tile's modes at once (fused pass, six waves / eight: 64x256x64 29.4 / 23.1 us,
    // 64x128x256 43.5 / 36.8; at other lengths the registers spill or it makes no difference)
    static constexpr int NW = sizeof(T) == 4 && N >= 128 && N % 3 != 0 ? 8 : 6, NT = NW * 64;
    // one empty row after every R0 positions (power of two) or every 4: the stores of the
    // first stage, R0 positions apart, then fall in different banks
    static constexpr int sk() {
        if (N % 3 == 0) return B < 16 ? 2 : 0;
        int k = 0;
        while ((1 << k) < P::R[0]) ++k;
        return B * (int)sizeof(cpx<T>) < 128 ? k : 0;
    }
    static constexpr int SK = sk();
    static constexpr int ROWS = SK ? N + ((N - 1) >> SK) : N, PLANE = ROWS * B;
    static __host__ __device__ constexpr int row(int pos) { return SK ? pos + (pos >> SK) : pos; }
    static constexpr int lds_bytes = (6 * PLANE + N * TwParts<T>::value) * (int)sizeof(cpx<T>);
    static constexpr bool PERSIST = lds_bytes > 80 * 1024;
    // waves per SIMD: six waves land on four SIMDs as 2, 2, 1, 1, so two workgroups need four
    static constexpr int WAVES = PERSIST ? 2 : 4;
};

// A column of one component's plane; its lanes lie in one wave.
template <typename T, class C>
struct TileCol {
    cpx<T>* p;
    __device__ __forceinline__ void st(int pos, cpx<T> a) { p[C::row(pos) * C::B] = a; }
    __device__ __forceinline__ cpx<T> ld(int pos) const { return p[C::row(pos) * C::B]; }
    __device__ __forceinline__ void sync() { wave_lds_sync(); }
    __device__ __forceinline__ void after_load() { wave_lds_sync(); }
};

// Modes, launch geometry and partial records as k_fused along y (AXIS = 1).
template <typename T, class P, int MODE>
__global__ void __launch_bounds__((WideCfg<T, P>::NT), (WideCfg<T, P>::WAVES))
k_fused_wide(const MemberDesc<T>* __restrict__ md, int M, int n_outer, int ntx, long pstride, long ostride, long cs,
             const cpx<T>* __restrict__ tw, int want_inv) {
    using C = WideCfg<T, P>;
    constexpr int N = P::N, E = P::E, TT = P::T, B = C::B, NT = C::NT, PLANE = C::PLANE;
    constexpr int Q = NQ<MODE>::value;
    // values of the next tile loaded before the modes; the others after the inverse
    // transform, where all 16 FP64 values of length 256 beside the transform's would spill
    // (fused pass of 256^3: all early 480 us, half 378, a quarter 406)
    constexpr int kEarly = N == 256 && sizeof(T) == 8 && (MODE == Z_STEP || MODE == Z_JUMP) ? E / 2 : E;
    __shared__ cpx<T> s_x[6 * PLANE];
    __shared__ cpx<T> s_tw[N * TwParts<T>::value];
    __shared__ double s_red[(NT / 64) * Q];
    const MemberDesc<T>& mem = md[blockIdx.z];
    const PropParams pp = mem.pp;
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6), lane = (int)threadIdx.x & 63;
    // with eight waves, two idle in the transforms: 0 and 1 or 2 and 3, by turns of the eight
    // workgroups that go to the eight XCDs
    const int idle = C::NW == 8 ? (((int)blockIdx.x >> 3) & 1) * 2 : 0;
    const int qw = C::NW == 8 ? (wave < idle ? wave : wave - 2) : wave;
    const bool fft = C::NW != 8 || wave < idle || wave >= idle + 2;
    const int q = fft ? qw : 0, tc = lane % B, t = lane / B;
    const int G = (int)gridDim.x, ntiles = ntx * n_outer;
    const unsigned cbytes = (unsigned)cs * sizeof(cpx<T>);
    const unsigned sstep = (unsigned)(TT * pstride) * sizeof(cpx<T>);
    const __amdgpu_buffer_rsrc_t rs = make_rsrc((MODE == Z_JUMP ? mem.spec : mem.work) + q * cs, cbytes);
    const __amdgpu_buffer_rsrc_t rd = make_rsrc(mem.work + q * cs, cbytes);
    auto voff_of = [&](int w, bool& active) {
        const int col = (w % ntx) * B + tc;
        active = col < M;
        return (unsigned)(t * pstride + (w / ntx) * ostride + (active ? col : M - 1)) * sizeof(cpx<T>);
    };
    // the waves in the order in which they take the modes: with six waves on four SIMDs,
    // the two that share no SIMD with another come first
    const int slot = (C::NW == 8 ? wave : (wave + 4) % 6) * 64 + lane;
    TileCol<T, C> lds{s_x + q * PLANE + tc};

    double acc[Q];
#pragma unroll
    for (int i = 0; i < Q; ++i) acc[i] = 0.0;
    int k = 0, w = persist_tile(0, G);
    bool active;
    unsigned voff = voff_of(w < ntiles ? w : 0, active);
    cpx<T> nv[E];
    if (fft) load_col<T, P>(nv, rs, voff, sstep);
    stage_table_plan<P>(s_tw, tw);
    __syncthreads();
    while (w < ntiles) {  // uniform over the workgroup
        const int wn = C::PERSIST ? persist_tile(k + 1, G) : ntiles;
        bool nactive = false;
        unsigned nvoff = 0;
        if (fft) {
            cpx<T> v[E];
#pragma unroll
            for (int i = 0; i < E; ++i) v[i] = nv[i];
            if constexpr (MODE != Z_JUMP) {
                fft_pencil<P, false, kStagedTw>(v, t, lds, s_tw);
                lds.after_load();
            }
#pragma unroll
            for (int i = 0; i < E; ++i) lds.st(t + TT * (MODE == Z_JUMP ? m_first<P>(i) : m_last<P>(i)), v[i]);
        }
        __syncthreads();
        if (C::PERSIST && wn < ntiles) {
            nvoff = voff_of(wn, nactive);
#pragma unroll
            for (int i = 0; i < kEarly; ++i) nv[i] = BufIO<T>::ld(rs, nvoff, (unsigned)m_first<P>(i) * sstep);
        }
        // modes, in pairs ky and -ky, which share the phase and the coefficients (the
        // pair 0 is ky = 0 and the Nyquist index, both with Omega_y = 0): thread i takes
        // pairs i, i + NT, ... of the tile, all of one column
        {
            const int mc = slot % B, col = (w % ntx) * B + mc, o = w / ntx;
            const double bx = col == 0 ? 0.0 : pp.nu[0] * (double)col;  // packed column: Omega_x = 0 at 0 and Nx/2
            const double bz = omega(o, n_outer, pp.nu[2]);
            const double wt = col == 0 ? 1.0 : 2.0;
            const bool sum = want_inv && col < M;
            constexpr bool kPencil = Q == INV_NPART;
            constexpr bool kProp = MODE == Z_STEP || MODE == Z_JUMP;
            PencilSums ps;
#pragma unroll 1
            for (int m = slot; m < N / 2 * B; m += NT) {
                const int kp = m / B;
                const double by0 = pp.nu[1] * (double)kp;
                PropCoef<T> pc;
                if constexpr (kProp) pc = prop_coef<T>(bx, by0, bz, pp);
#pragma unroll
                for (int half = 0; half < 2; ++half) {
                    const int ky = half == 0 ? kp : (kp == 0 ? N / 2 : N - kp);
                    const double by = half == 0 ? by0 : -by0;
                    cpx<T>* at = s_x + C::row(ky) * B + mc;
                    cpx<T> h[3] = {at[0], at[PLANE], at[2 * PLANE]};
                    cpx<T> e[3] = {at[3 * PLANE], at[4 * PLANE], at[5 * PLANE]};
                    if constexpr (kProp) {
                        if (half == 1) mirror_y(pc);
                        prop_apply(h, e, pc);
                    } else {
                        const T s = (T)pp.inv_ns;
#pragma unroll
                        for (int c = 0; c < 3; ++c) {
                            h[c] = scale(h[c], s);
                            e[c] = scale(e[c], s);
                        }
                    }
                    if (sum) {
                        if constexpr (kPencil) ps.add(bx, by, bz, h, e);
                        else accumulate_invariants<Q>(acc, wt, bx, by, bz, h, e, pp);
                    }
                    if constexpr (kProp) {
#pragma unroll
                        for (int c = 0; c < 3; ++c) {
                            at[c * PLANE] = h[c];
                            at[(3 + c) * PLANE] = e[c];
                        }
                    }
                    __builtin_amdgcn_sched_barrier(0);  // one mode's temporaries live at a time
                }
            }
            if constexpr (kPencil) {
                if (sum) {
                    double a[INV_NPART];
                    ps.finish(a, wt, bx, bz, pp);
#pragma unroll
                    for (int i = 0; i < INV_NPART; ++i) acc[i] += a[i];
                }
            }
        }
        __syncthreads();
        if constexpr (MODE == Z_STEP || MODE == Z_JUMP) if (fft) {
            cpx<T> v[E];
#pragma unroll
            for (int i = 0; i < E; ++i) v[i] = lds.ld(t + TT * m_first<P>(i));
            lds.after_load();
            fft_pencil<P, true, kStagedTw>(v, t, lds, s_tw);
            if (C::PERSIST && wn < ntiles) {
#pragma unroll
                for (int i = kEarly; i < E; ++i) nv[i] = BufIO<T>::ld(rs, nvoff, (unsigned)m_first<P>(i) * sstep);
            }
            store_col<T, P, EIFP_FUSED_ST_AUX>(v, rd, voff, sstep, active);
        }
        ++k;
        w = wn;
        voff = nvoff;
        active = nactive;
    }
    if (want_inv) block_reduce_store<NT, Q>(acc, mem.partials + (long)blockIdx.x * Q, s_red);
}

}  // namespace eifp
