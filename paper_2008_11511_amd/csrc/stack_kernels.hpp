// stack_kernels.hpp - the frame-size templated kernels of one stack: the row
// passes, the column pass and the plain batched FFT.  Each frame size is
// instantiated in a translation unit of its own (inst_N.hip).
#pragma once

#include "common.hpp"

namespace ptycho {

// ============================================================ row passes ===

// Frames whose same rows neighbouring blocks of a row pass take (row_block); 0:
// the rows of one frame after another, the frame a value of each thread.
// What a frame of 512 points reads besides its waves - view and probe, the
// line search's two directions too - is 4 to 8 MB per mode, more than an
// XCD's 4 MB L2 holds from one frame to the next, and eight frames side by side
// read a probe row once: rows of 400 frames x 4 modes 895 -> 823 us, the line
// search's 3203 -> 1764 us; the DM form, which streams old waves as well, is
// best at four (1611 -> 1547 us, eight 1550-1680).  But a stack that the eight
// L2s hold together (32 MB) is read by the column pass from the L2 that its
// rows were written to, and only if an XCD's blocks are of few whole frames:
// intensities of 4 frames x 4 modes took 24.6 us in the frames' order and 28.5
// side by side, 8 frames x 1 mode 15.4 and 18.9; of 8 frames x 4 modes (64 MB)
// 42.8 and 37.0.  So side_frames() gives 1 up to there.
// At 256 and 1024 points, and at 2048 in the plain form, the gain is the frame's
// index being one per block (scalar view and probe bases), in the frames' order:
// intensities of 256 frames of 256^2 x 4 modes 228 -> 222 us, of 64 frames of
// 1024^2 x 1 628 -> 472 us, of 4 frames of 2048^2 x 4 574 -> 512 us.  The DM
// form loses by it at 256 (256 frames x 4 modes 825 -> 844 us a cycle) and 2048
// points.  The line search at 1024 points gains by four frames side by side in
// the near field (17 frames x 4 modes 2412 -> 1578 us) and where the third
// transform is kept (16 frames x 4 modes 2591 -> 2469 us a ML cycle), but loses
// where the far field forms all three (32 frames x 2 modes: 1306 us in the
// frames' order, 1742 side by side, 1385 with a scalar index alone).
template <int N, int MODE, bool NF>
__host__ __device__ constexpr int fwd_frames() {
    if (N == 256) return MODE == IN_PHI ? 1 : 0;
    if (N == 512) return MODE == IN_DM ? 4 : 8;
    if (N == 1024) return MODE == IN_LS ? (NF ? 4 : 0) : MODE == IN_LS2 ? 4 : 1;
    return N > 1024 && MODE == IN_PHI ? 1 : 0;
}
// The frames side by side of a launch of S frames x K modes, up to fwd_frames.
template <int N, int MODE, bool NF>
static int side_frames(int S, int K) {
    const size_t bytes = sizeof(float2) * S * K * N * N;
    return N == 512 && MODE == IN_PHI && bytes <= (size_t(32) << 20) ? 1 : fwd_frames<N, MODE, NF>();
}
// Measured to gain at 512 points with four modes only: 1553 -> 1439 us (AP, 400
// frames), 1693 -> 1611 us (DM); with three modes 451 -> 481 us, at 1024 points,
// whatever the modes, up to 40% slower.
template <int N, int K>
__host__ __device__ constexpr int inv_frames() {
    return N == 512 && K >= 4 ? 4 : 0;
}

// Forward row FFT of the stack's exit waves.  Block = RB consecutive rows of
// the flattened (slot, y) row index of one probe mode (blockIdx.y), or RB rows
// of one frame in row_block's order; thread = (row, t).  The object view is re-read per mode from the caches.
template <int N, int MODE, bool NF, bool SUB>
__global__ __launch_bounds__(256) void k_rows_fwd(StackArgs a) {
    using G = RowGeom<N>;
    constexpr int E = G::E, T = G::T, RB = G::RB, FR = fwd_frames<N, MODE, NF>();
    __shared__ float2 lds[G::LDS_F2];
    const int tid = threadIdx.x, rr = tid / T, t = tid % T;
    const int k = blockIdx.y;
    int s, y;
    bool active = true;
    if constexpr (FR > 0) {
        const int2 b = row_block<N, RB>(xcd_block(blockIdx.x, gridDim.x), a.S, FR > 1 ? a.side : 1);
        s = b.x;
        y = b.y + rr;
    } else {
        const int g = xcd_block(blockIdx.x, gridDim.x) * RB + rr;
        active = g < a.S * N;
        const int gg = active ? g : a.S * N - 1;
        s = gg / N;
        y = gg % N;
    }
    const int j = a.order[a.s0 + s];
    const int2 o = a.offs[j];
    const size_t orow = (size_t)(o.x + y) * a.Nx + o.y;
    RowLds<N> L(lds, rr);
    // line search: A = P O, B = P dO + dP O, C = dP dO; IN_LS2 forms B and C
    // only (A is the gradient pass's kept row transform)
    constexpr bool LSM = (MODE == IN_LS) || (MODE == IN_LS2);
    constexpr int SETS = (MODE == IN_LS) ? 3 : (MODE == IN_LS2) ? 2 : 1;
    const float2 *prow = a.probe + ((size_t)k * N + y) * N;
    const float2 *drow = LSM ? a.dprobe + ((size_t)k * N + y) * N : nullptr;
    // The three line-search rows held together need 3E complex registers;
    // at 2048 points each set is formed and transformed on its own instead
    // (the object and probe rows are read again, from the caches).
    constexpr bool SPLIT = LSM && N >= 2048;
    float2 u[SPLIT ? 1 : SETS][E];
    // the object view (and the line search's direction view) at column x:
    // integer windows read the row, sub-pixel windows (SUB) interpolate
    ViewRow vr{};
    if constexpr (SUB) vr = view_row(a.Ny, a.Nx, o, a.frac[j], y);
#pragma unroll
    for (int set = 0; set < SETS; ++set) {
        const int sl = SPLIT ? 0 : set;
        auto fill = [&](auto view) {
#pragma unroll
            for (int e = 0; e < E; ++e) {
                const int x = in_index<N, E, -1>(t, e);
                const float2 ov = view(a.obj, x);
                const float2 p = prow[x];
                if constexpr (SPLIT) {
                    const float2 dv = view(a.dobj, x), dp = drow[x];
                    const int q = (MODE == IN_LS2) ? set + 1 : set;
                    u[0][e] = q == 0 ? cmul(ov, p) : q == 1 ? cadd(cmul(dv, p), cmul(ov, dp)) : cmul(dv, dp);
                } else if constexpr (MODE == IN_LS2) {
                    const float2 dv = view(a.dobj, x);
                    const float2 dp = drow[x];
                    u[0][e] = cadd(cmul(dv, p), cmul(ov, dp));
                    u[1][e] = cmul(dv, dp);
                } else if constexpr (MODE == IN_LS) {
                    const float2 dv = view(a.dobj, x);
                    const float2 dp = drow[x];
                    u[0][e] = cmul(ov, p);
                    u[1][e] = cadd(cmul(dv, p), cmul(ov, dp));
                    u[2][e] = cmul(dv, dp);
                } else if constexpr (MODE == IN_DM) {
                    const float2 phi = cmul(ov, p);
                    // the old exit waves are read once: non-temporal
                    const float2 ps = ld_stream(a.psi + (((size_t)j * a.K + k) * N + y) * N + x);
                    u[0][e] = make_float2(2.0f * phi.x - ps.x, 2.0f * phi.y - ps.y);
                } else {
                    u[0][e] = cmul(ov, p);
                }
            }
        };
        if (SPLIT || set == 0) {
            if constexpr (SUB) fill([&](const float2 *b, int x) { return view_at(b, vr, x); });
            else fill([&](const float2 *b, int x) { return b[orow + x]; });
        }
        const int tt = SPLIT ? opaque(t) : t;
        fft1d<N, E, -1>(u[sl], tt, L);
        if constexpr (NF) {
            // Dx: the x factor of the transfer function, then back to x
            const float2 *qx = a.prop + N;
            const int t1 = opaque(tt);
#pragma unroll
            for (int e = 0; e < E; ++e) u[sl][e] = cmul(u[sl][e], qx[out_index<N, E, -1>(t1, e)]);
            fft1d<N, E, +1>(u[sl], t1, L);
        }
        float2 *dst = (MODE == IN_PHI ? a.fwd : a.scr) + ((size_t)s * SETS * a.K + set * a.K + k) * N * N;
        if (active) {
#pragma unroll
            for (int e = 0; e < E; ++e) {
                const int x = NF ? out_index<N, E, +1>(t, e) : out_index<N, E, -1>(t, e);
                st_stream(dst + scr_at<N>(y, x), u[sl][e]);
            }
        }
    }
}


// Inverse row FFT of the stack scratch and the real-space epilogue.  A block
// has TPM threads (whole wavefronts) per probe mode, all on the same RQ rows.
// Outputs:
// OUT_SCR the exit waves back into the scratch, OUT_STORE into psi_out
// [J][K][N][N], OUT_DM Phi + u into psi_out, OUT_NONE nothing.  With WQ the
// block also writes q = sum_k conj(P_k) Psi_k (the modes summed through LDS),
// the frame's term of the object numerator, to qbuf, so that the object
// gather reads one plane per frame instead of K exit waves and K probe
// values.
template <int N, int K, int MODE, bool WQ, bool NF, bool SUB>
__global__ __launch_bounds__(InvRowGeom<N>::TPM * K) void k_rows_inv(StackArgs a) {
    using G = InvRowGeom<N>;
    constexpr int E = G::E, T = G::T, RQ = G::RQ, FR = inv_frames<N, K>();
    __shared__ float2 lds[K * RQ * G::ROW_F2];
    const int k = threadIdx.x / G::TPM, lane = threadIdx.x % G::TPM, rr = lane / T, t = lane % T;
    int s, y;
    bool active = true;
    if constexpr (FR > 0) {
        const int2 b = row_block<N, RQ>(xcd_block(blockIdx.x, gridDim.x), a.S, FR);
        s = b.x;
        y = b.y + rr;
    } else {
        const int g = xcd_block(blockIdx.x, gridDim.x) * RQ + rr;
        active = g < a.S * N;
        const int gg = active ? g : a.S * N - 1;
        s = gg / N;
        y = gg % N;
    }
    const int j = a.order[a.s0 + s];
    RowLds<N> L(lds, k * RQ + rr);

    float2 *src = a.scr + ((size_t)s * K + k) * N * N;
    float2 u[E];
#pragma unroll
    for (int e = 0; e < E; ++e)          // read once: non-temporal, the caches keep the views and the probe
        u[e] = ld_stream(src + scr_at<N>(y, NF ? in_index<N, E, -1>(t, e) : in_index<N, E, +1>(t, e)));
    if constexpr (NF) {
        // Dx^-1: forward transform, the conjugate x factor, inverse below
        fft1d<N, E, -1>(u, t, L);
        const float2 *qx = a.prop + N;
#pragma unroll
        for (int e = 0; e < E; ++e) u[e] = cmulc(qx[out_index<N, E, -1>(t, e)], u[e]);
    }
    const float2 *prow = a.probe + ((size_t)k * N + y) * N;
    const size_t prow_psi = (((size_t)j * K + k) * N + y) * N;
    size_t orow = 0;
    if constexpr (MODE == OUT_DM) {
        const int2 o = a.offs[j];
        orow = (size_t)(o.x + y) * a.Nx + o.y;
    }
    ViewRow vr{};
    if constexpr (SUB) vr = view_row(a.Ny, a.Nx, a.offs[j], a.frac[j], y);
    // The DM form loads the object view and the probe row before the
    // transform, so that their latency overlaps its passes (loads cannot move
    // across the transform's barriers): measured 10% faster at 256 points
    // with 3 modes and 22% at 512 with 4.  Sub-pixel views (four object
    // values per pixel) and the near field would hold too many registers.
    constexpr bool PF = MODE == OUT_DM && !NF && !SUB;
    constexpr bool PP = PF;
    float2 ovp[PF ? E : 1], pvp[PP ? E : 1];
#pragma unroll
    for (int e = 0; e < E; ++e) {
        const int x = out_index<N, E, +1>(t, e);
        if constexpr (PF) ovp[e] = SUB ? view_at(a.obj, vr, x) : a.obj[orow + x];
        if constexpr (PP) pvp[e] = prow[x];
    }
    fft1d<N, E, +1>(u, t, L);
    float2 qk[E];
#pragma unroll
    for (int e = 0; e < E; ++e) {
        const int x = out_index<N, E, +1>(t, e);
        float2 v = u[e];
        float2 pe;
        if constexpr (PP) pe = pvp[e];
        else pe = prow[x];
        if constexpr (MODE == OUT_DM) {
            float2 oe;
            if constexpr (PF) oe = ovp[e];
            else oe = SUB ? view_at(a.obj, vr, x) : a.obj[orow + x];
            if (active) v = cadd(cmul(oe, pe), v);
        }
        if (active) {
            if constexpr (MODE == OUT_SCR) src[scr_at<N>(y, x)] = v;
            if constexpr (MODE == OUT_STORE || MODE == OUT_DM) st_stream(a.psi_out + prow_psi + x, v);
        }
        if constexpr (WQ) qk[e] = cmulc(pe, v);
    }
    if constexpr (WQ && K == 1) {        // the frame's term is this thread's own
        if (active) {
            float2 *qrow = a.qbuf + ((size_t)s * N + y) * N;
#pragma unroll
            for (int e = 0; e < E; ++e) st_stream(qrow + out_index<N, E, +1>(t, e), qk[e]);
        }
    } else if constexpr (WQ) {
        __syncthreads();                 // the transforms' LDS reads are done
#pragma unroll
        for (int e = 0; e < E; ++e) L.st(out_index<N, E, +1>(t, e), qk[e]);
        __syncthreads();
        // the threads of mode k sum and write the pixels of their elements
        // e = k, k + K, ...
        if (active) {
            float2 *qrow = a.qbuf + ((size_t)s * N + y) * N;
#pragma unroll
            for (int e = 0; e < E; ++e) {
                if (e % K != k) continue;
                const int x = out_index<N, E, +1>(t, e);
                float2 q = RowLds<N>(lds, rr).ld(x);
#pragma unroll
                for (int m = 1; m < K; ++m) q = cadd(q, RowLds<N>(lds, m * RQ + rr).ld(x));
                st_stream(qrow + x, q);
            }
        }
    }
}

// Inverse row FFT of the gradient pass with both sums taken from the gradient
// waves in registers: a block walks the frames of its consecutive chunks
// (C blocks per row group, M chunks in all, M >= C) on the same RQ rows, writes
// each frame's q as above, and keeps a chunk's probe numerators
// sum_j conj(O_j) psi_jk and denominators sum_j |O_j|^2 of its rows, which
// k_probe_reduce adds over the chunks.  Integer windows.
// M is separate from C so that a chunk, a running sum in 32 bits, is as short
// as the sums need while the blocks are as many as the chip takes.
// Bound by memory; it reads K and writes one complex frame where k_rows_inv
// also wrote the K waves back and k_gather_probe read them again: 500 frames
// of 256^2 x 3 modes took 347 + 152 us and take 331, 400 of 512^2 x 4 1552 +
// 601 and take 1690, 1000 of 128^2 x 4 353 + 102 and take 238.  The sums cost
// 200-255 registers, two waves per SIMD; held to three, the spills cost more
// than the third wave gives (256^2 x 3: 493 us).  With one mode the compiler
// would reach for three by itself and load less at a time: 17 near-field frames
// of 512^2 55 us, 36 when held to two, 17 of 1024^2 209 and 186; with more
// modes, or at 2048 points, the hint makes the code worse (512^2 x 4: 1758).
// The view is loaded after the transform, which the registers then need not
// hold (512 x 1: 430 against 506 us), except at 2048 points, where the probe and
// view rows no longer stay in the L2 from one frame to the next (20 frames: 586
// against 732).
template <int N, int K, bool NF>
__global__ __launch_bounds__(InvRowGeom<N>::TPM * K)
__attribute__((amdgpu_waves_per_eu(2, N < 2048 && K == 1 ? 2 : 8)))
void k_rows_inv_grad(StackArgs a, int C, int M, float2 *pnum, float *pden) {
    using G = InvRowGeom<N>;
    constexpr int E = G::E, T = G::T, RQ = G::RQ, RG = N / RQ;
    static_assert(N % RQ == 0, "a block's rows are of one frame");
    constexpr bool EARLY = N >= 2048;    // load the view before the transform
    __shared__ float2 lds[K * RQ * G::ROW_F2];
    const int k = threadIdx.x / G::TPM, lane = threadIdx.x % G::TPM, rr = lane / T, t = lane % T;
    const int b = xcd_block(blockIdx.x, gridDim.x), c = b / RG, y = b % RG * RQ + rr;
    const int m0 = (int)((long)c * M / C), m1 = (int)((long)(c + 1) * M / C);
    RowLds<N> L(lds, k * RQ + rr);
    const float2 *prow = a.probe + ((size_t)k * N + y) * N;
    const size_t n2 = (size_t)N * N;
    for (int m = m0; m < m1; ++m) {
        const int s0 = (int)((long)m * a.S / M), s1 = (int)((long)(m + 1) * a.S / M);
        float2 acc[E];
        float den[E];
#pragma unroll
        for (int e = 0; e < E; ++e) {
            acc[e] = make_float2(0.0f, 0.0f);
            den[e] = 0.0f;
        }
        for (int s = s0; s < s1; ++s) {
            const int2 o = a.offs[a.order[a.s0 + s]];
            const float2 *src = a.scr + ((size_t)s * K + k) * N * N;
            const float2 *orow = a.obj + ((size_t)(o.x + y) * a.Nx + o.y);
            const int tf = opaque(t);
            float2 u[E], ov[E];
#pragma unroll
            for (int e = 0; e < E; ++e)
                u[e] = ld_stream(src + scr_at<N>(y, NF ? in_index<N, E, -1>(tf, e) : in_index<N, E, +1>(tf, e)));
            if constexpr (EARLY) {
#pragma unroll
                for (int e = 0; e < E; ++e) ov[e] = orow[out_index<N, E, +1>(tf, e)];
            }
            if constexpr (NF) {
                fft1d<N, E, -1>(u, tf, L);
                const float2 *qx = a.prop + N;
#pragma unroll
                for (int e = 0; e < E; ++e) u[e] = cmulc(qx[out_index<N, E, -1>(tf, e)], u[e]);
            }
            const int t1 = NF ? opaque(tf) : tf;
            fft1d<N, E, +1>(u, t1, L);
            if constexpr (!EARLY) {
#pragma unroll
                for (int e = 0; e < E; ++e) ov[e] = orow[out_index<N, E, +1>(t1, e)];
            }
#pragma unroll
            for (int e = 0; e < E; ++e) {
                const float2 cv = cmulc(ov[e], u[e]);
                acc[e] = cadd(acc[e], cv);
                if (e % K == k) den[e] += cnorm(ov[e]);
                u[e] = cmulc(prow[out_index<N, E, +1>(t1, e)], u[e]);
            }
            float2 *qrow = a.qbuf + ((size_t)s * N + y) * N;
            if constexpr (K == 1) {
#pragma unroll
                for (int e = 0; e < E; ++e) st_stream(qrow + out_index<N, E, +1>(t1, e), u[e]);
            } else {
                __syncthreads();             // the transforms' LDS reads are done
#pragma unroll
                for (int e = 0; e < E; ++e) L.st(out_index<N, E, +1>(t1, e), u[e]);
                __syncthreads();
#pragma unroll
                for (int e = 0; e < E; ++e) {
                    if (e % K != k) continue;
                    const int x = out_index<N, E, +1>(t1, e);
                    float2 q = RowLds<N>(lds, rr).ld(x);
#pragma unroll
                    for (int h = 1; h < K; ++h) q = cadd(q, RowLds<N>(lds, h * RQ + rr).ld(x));
                    st_stream(qrow + x, q);
                }
            }
        }
        float2 *pn = pnum + ((size_t)m * K + k) * n2 + (size_t)y * N;
        float *pd = pden + (size_t)m * n2 + (size_t)y * N;
#pragma unroll
        for (int e = 0; e < E; ++e) {
            const int x = out_index<N, E, +1>(t, e);
            pn[x] = acc[e];
            if (e % K == k) pd[x] = den[e];
        }
    }
}

// ========================================================== column pass ===
// OP_CORR writes (s - 1) F(X) instead of s F(X): since P_F(X) = X + F^-1((s-1) F(X))
// (s = 1 at bad pixels), the DM update Psi + P_F(2 Phi - Psi) - Phi equals
// Phi + F^-1((s - 1) F(2 Phi - Psi)), which the inverse row pass forms from the
// views alone, without reading the old exit waves again.

// Exchange buffers of the read-only column pass: the line search's three
// transforms of a mode run pass by pass together while their buffers fit
// 96 KiB of LDS, one after the other through one buffer beyond that.
template <int N, int OP, bool NF = false>
struct ColSeqBufs {
    static constexpr int SETS = (OP == OP_LS || OP == OP_LS2) ? 3 : 1;
    using G = ColGeom<N, seq_cb(N, SETS == 3)>;
    static constexpr int value = ((size_t)SETS * ColGeom<N>::LDS_F2 * 8 <= 96 * 1024) ? SETS : 1;
    // waves per SIMD: the far-field LLK and intensities need 81 to 85 registers,
    // one to five too many for six waves, and fit 80 with at most one spilled
    // (LLK of 60 frames of 512^2 x 2 modes 172 -> 163 us)
    static constexpr int MIN_WAVES = !NF && SETS == 1 && N >= 128 && N <= 512 && (N != 256 || OP == OP_LLK) ? 6 : 1;
};

// Waves per SIMD a column kernel is compiled for: up to 3 modes the DM and
// gradient forms fit 128 registers without spilling and the 512-point
// projection with 12 bytes of spill, which gives 4 waves instead of 3 (two
// 512-thread blocks instead of one at 512 points, 3 modes: AP columns of 150
// frames 533 -> 362 us); the 256-point, 3-mode projection would spill 56 bytes
// and is faster at 3 waves (299 against 364 us, 500 frames).  The near-field
// pass at 2048 points with one mode gets 4 waves too, the 256-point, 4-mode
// projection 3 (two registers spilled; 170 registers would leave it 2: columns
// of a 100-frame AP cycle of 191 us 24 us slower).  The others are held to two
// waves: left alone, the compiler gives the 256-thread blocks of the 2048-point
// pass with three and four modes more than 256 registers, one wave per SIMD (AP
// cycle of 17 near-field frames, 4 modes: 6.44 ms, 5.01 held to two waves and 5.69
// in whole tiles).
template <int N, int K, int OP, bool NF>
struct ColMinWaves {
    static constexpr int value = ((!NF && ColJoint<N, K>::SEQ && N <= 512 && K <= 3 && (N == 512 || OP != OP_PROJECT)) ||
                                  (NF && N >= 2048 && K == 1)) ? 4
                                 : (!NF && N == 256 && K == 4 && OP == OP_PROJECT) ? 3 : 2;
};

// Row (y) index of register e of thread t at the detector-plane step: after
// the forward transform in the far field (a frequency), after the forward
// and inverse transforms in the near field (a pixel).
template <int N, int E, bool NF>
__device__ __forceinline__ int det_row(int t, int e) {
    return NF ? in_index<N, E, -1>(t, e) : out_index<N, E, -1>(t, e);
}

// The column transforms of all K modes, forward (DIR -1) or inverse (+1):
// joint pass by pass, or one mode after the other through one buffer.
template <int N, int E, int DIR, int K, bool SEQ, class Lds>
__device__ __forceinline__ void col_transforms(float2 (&u)[K][E], int t, Lds *L) {
    if constexpr (SEQ) {
        __syncthreads();     // earlier transforms' last LDS reads are done
#pragma unroll
        for (int k = 0; k < K; ++k) fft1d<N, E, DIR>(u[k], t, L[k]);
    } else {
        fftk<N, E, DIR, K>(u, t, L);
    }
}

// Near field: multiply the column spectra by Qy (CONJ: its conjugate).
template <int N, int E, int K, int NSET, bool CONJ>
__device__ __forceinline__ void apply_qy(float2 (&u)[K][E], const float2 *qy, int t) {
#pragma unroll
    for (int e = 0; e < E; ++e) {
        const float2 w = qy[out_index<N, E, -1>(t, e)];
#pragma unroll
        for (int k = 0; k < NSET; ++k) u[k][e] = CONJ ? cmulc(w, u[k][e]) : cmul(u[k][e], w);
    }
}

// Column FFTs of all K modes held together in registers, the Fourier-space
// step and (project / grad) the inverse column FFTs, written back in place.
template <int N, int K, int OP, bool NF>
__global__ __launch_bounds__((ColJoint<N, K>::G::THREADS), (ColMinWaves<N, K, OP, NF>::value)) void k_cols_joint(StackArgs a) {
    using G = typename ColJoint<N, K>::G;
    constexpr int E = G::E, CB = G::CB;
    extern __shared__ float2 lds_dyn[];
    const int tid = threadIdx.x, cl = tid % CB, t = tid / CB;
    const int blk = xcd_block(blockIdx.x, gridDim.x);
    const int g = blk * CB + cl;
    const bool active = g < a.S * N;
    const int gg = active ? g : a.S * N - 1;
    const int s = gg / N, c = gg % N;
    const int j = a.order[a.s0 + s];
    constexpr bool SEQ = ColJoint<N, K>::SEQ;
    ColLds<N, CB> L[K];
#pragma unroll
    for (int k = 0; k < K; ++k) L[k] = ColLds<N, CB>(lds_dyn + (SEQ ? 0 : k) * G::LDS_F2, cl);
    // far field: the unitary 1/N^2 of the forward and inverse 2D transforms;
    // near field: folded into the transfer-function factors
    constexpr float nrm = NF ? 1.0f : 1.0f / ((float)N * (float)N);

    // far field from 512 points (two waves per SIMD, latency-bound) the stack
    // is read non-temporally: 4000 x 512^2 x 4 modes, columns 25.2 -> 23.8 ms
    // per DM cycle; at 256 points it made the pass 5% slower
    // (not for half tiles: the other half of a line goes to another block)
    constexpr bool NT = !NF && N >= 512 && CB == ScrTile<N>::W;
    float2 u[K][E];
#pragma unroll
    for (int k = 0; k < K; ++k) {
        const float2 *src = a.colin + ((size_t)(s * K + k) * N) * N + scr_at<N>(0, c);
#pragma unroll
        for (int e = 0; e < E; ++e) {
            const float2 *at = src + in_index<N, E, -1>(t, e) * ScrTile<N>::W;
            u[k][e] = NT ? ld_stream(at) : *at;
        }
    }
    // the data of the pixels this thread will own after the transform are
    // loaded now: loads cannot move across the transform's barriers
    const float *io = a.iobs + (size_t)j * N * N + c;
    const unsigned bad_bits = mask_bits<E>(a.mask, [&](int e) { return det_row<N, E, NF>(t, e) * N + c; });
    float iobv[E];
#pragma unroll
    for (int e = 0; e < E; ++e) iobv[e] = io[(size_t)det_row<N, E, NF>(t, e) * N];
    col_transforms<N, E, -1, K, SEQ>(u, t, L);
    if constexpr (NF) {
        // Dy: to the detector plane
        const int t1 = opaque(t);
        apply_qy<N, E, K, K, false>(u, a.prop, t1);
        col_transforms<N, E, +1, K, SEQ>(u, t1, L);
    }

    float in[E];
#pragma unroll
    for (int e = 0; e < E; ++e) {
        in[e] = 0.0f;
#pragma unroll
        for (int k = 0; k < K; ++k) in[e] += cnorm(u[k][e]);
        in[e] *= nrm;
    }
    // the background (L2-resident, usually absent) is read here rather than
    // with Iobs, so that it holds no registers across the transform
    if (a.bg != nullptr) {
#pragma unroll
        for (int e = 0; e < E; ++e) in[e] += a.bg[det_row<N, E, NF>(t, e) * N + c];
    }
    double acc = 0.0;
#pragma unroll
    for (int e = 0; e < E; ++e) {
        const float inten = in[e];
        const bool bad = (bad_bits >> e) & 1u;
        const float iob = iobv[e];
        float sc;
        if constexpr (OP == OP_PROJECT) {
            const float r = iob / fmaxf(inten, a.eps);
            sc = bad ? nrm : sqrtf(r) * nrm;
            if (a.s2 != nullptr && active) a.s2[((size_t)s * N + det_row<N, E, NF>(t, e)) * N + c] = bad ? 1.0f : r;
        } else if constexpr (OP == OP_CORR) {
            sc = bad ? 0.0f : (sqrtf(iob / fmaxf(inten, a.eps)) - 1.0f) * nrm;
        } else {
            const float ifl = fmaxf(inten, a.eps);
            sc = bad ? 0.0f : (1.0f - iob / ifl) * nrm;
            if (!bad && active) acc += (double)llk_term(ifl, iob);
        }
#pragma unroll
        for (int k = 0; k < K; ++k) u[k][e] = cscale(u[k][e], sc);
    }
    const int t3 = NF ? opaque(t) : t;
    if constexpr (NF) {
        // Dy^-1: back from the detector plane (the inverse transform below)
        const int t2 = opaque(t);
        col_transforms<N, E, -1, K, SEQ>(u, t2, L);
        apply_qy<N, E, K, K, true>(u, a.prop, t2);
    }
    col_transforms<N, E, +1, K, SEQ>(u, t3, L);
    if (active) {
#pragma unroll
        for (int k = 0; k < K; ++k) {
            float2 *dst = a.scr + ((size_t)(s * K + k) * N) * N + scr_at<N>(0, c);
#pragma unroll
            for (int e = 0; e < E; ++e) dst[out_index<N, E, +1>(t, e) * ScrTile<N>::W] = u[k][e];
        }
    }
    if constexpr (OP == OP_GRAD) {
        const double r = block_sum(acc);
        if (threadIdx.x == 0) a.red[blk] = r;
    }
}

// Column FFTs one mode at a time for the read-only Fourier-space steps:
// LLK, calculated intensity, and the line-search terms I0, I1, I2.  The
// transforms' inputs are read once, non-temporally (line search at 500 x
// 256^2 x 3 modes: ML cycle 2.34 -> 2.31 ms).
template <int N, int OP, bool NF>
__global__ __launch_bounds__((ColSeqBufs<N, OP>::G::THREADS), (ColSeqBufs<N, OP, NF>::MIN_WAVES))
void k_cols_seq(StackArgs a) {
    using G = typename ColSeqBufs<N, OP>::G;
    constexpr int E = G::E, CB = G::CB;
    extern __shared__ float2 lds_dyn[];
    const int tid = threadIdx.x, cl = tid % CB, t = tid / CB;
    const int blk = xcd_block(blockIdx.x, gridDim.x);
    const int g = blk * CB + cl;
    const bool active = g < a.S * N;
    const int gg = active ? g : a.S * N - 1;
    const int s = gg / N, c = gg % N;
    const int j = a.order[a.s0 + s];
    constexpr float nrm = NF ? 1.0f : 1.0f / ((float)N * (float)N);
    constexpr int SETS = ColSeqBufs<N, OP>::SETS;
    constexpr bool ONE_BUF = ColSeqBufs<N, OP>::value == 1 && SETS > 1;

    // whole tiles are read once; the other half of a half tile's lines goes to
    // another block
    auto ld_col = [](const float2 *p) { return CB == ScrTile<N>::W ? ld_stream(p) : *p; };
    float i0[E], i1[E], i2[E];
#pragma unroll
    for (int e = 0; e < E; ++e) i0[e] = i1[e] = i2[e] = 0.0f;
    // the SETS transforms of a mode run pass by pass together
    ColLds<N, CB> Ls[SETS];
#pragma unroll
    for (int set = 0; set < SETS; ++set) Ls[set] = ColLds<N, CB>(lds_dyn + (ONE_BUF ? 0 : set) * G::LDS_F2, cl);
    // set `set` of mode k: A from the kept row transforms (OP_LS2) or the
    // scratch, B and C from the scratch
    auto src_of = [&](int set, int k) -> const float2 * {
        if constexpr (OP == OP_LS2) {
            if (set == 0) return a.colin + ((size_t)(s * a.K + k) * N) * N + scr_at<N>(0, c);
            return a.scr + ((size_t)(s * 2 * a.K + (set - 1) * a.K + k) * N) * N + scr_at<N>(0, c);
        }
        return a.colin + ((size_t)(s * SETS * a.K + set * a.K + k) * N) * N + scr_at<N>(0, c);
    };
    for (int k = 0; k < a.K; ++k) {
        if constexpr (ONE_BUF) {
            // one transform at a time (large N): keep A, fold B and C into
            // the sums as soon as each is transformed
            float2 A[1][E], V[1][E];
            auto load_transform = [&](float2 (&v)[1][E], int set) {
                const float2 *src = src_of(set, k);
#pragma unroll
                for (int e = 0; e < E; ++e) v[0][e] = ld_col(src + in_index<N, E, -1>(t, e) * ScrTile<N>::W);
                const int t0 = opaque(t);
                col_transforms<N, E, -1, 1, false>(v, t0, Ls);
                if constexpr (NF) {
                    const int t1 = opaque(t);
                    apply_qy<N, E, 1, 1, false>(v, a.prop, t1);
                    col_transforms<N, E, +1, 1, false>(v, t1, Ls);
                }
            };
            load_transform(A, 0);
            load_transform(V, 1);
#pragma unroll
            for (int e = 0; e < E; ++e) {
                i0[e] += cnorm(A[0][e]);
                i1[e] += 2.0f * cmulc(A[0][e], V[0][e]).x;
                i2[e] += cnorm(V[0][e]);
            }
            load_transform(V, 2);
#pragma unroll
            for (int e = 0; e < E; ++e) i2[e] += 2.0f * cmulc(A[0][e], V[0][e]).x;
            continue;
        }
        float2 u[SETS][E];
#pragma unroll
        for (int set = 0; set < SETS; ++set) {
            const float2 *src = src_of(set, k);
#pragma unroll
            for (int e = 0; e < E; ++e) u[set][e] = ld_col(src + in_index<N, E, -1>(t, e) * ScrTile<N>::W);
        }
        col_transforms<N, E, -1, SETS, ONE_BUF>(u, t, Ls);
        if constexpr (NF) {
            const int t1 = opaque(t);
            apply_qy<N, E, SETS, SETS, false>(u, a.prop, t1);
            col_transforms<N, E, +1, SETS, ONE_BUF>(u, t1, Ls);
        }
#pragma unroll
        for (int e = 0; e < E; ++e) {
            i0[e] += cnorm(u[0][e]);
            if constexpr (OP == OP_LS || OP == OP_LS2) {
                const float2 ab = cmulc(u[0][e], u[1][e]);
                const float2 ac = cmulc(u[0][e], u[2][e]);
                i1[e] += 2.0f * ab.x;
                i2[e] += cnorm(u[1][e]) + 2.0f * ac.x;
            }
        }
    }
    const float *io = a.iobs + (size_t)j * N * N + c;
    // all data are loaded before the first are used
    float iobv[E];
    unsigned bad_bits = 0;
#pragma unroll
    for (int e = 0; e < E; ++e) {
        i0[e] *= nrm;
        if constexpr (OP != OP_ICALC) iobv[e] = io[(size_t)det_row<N, E, NF>(t, e) * N];
    }
    if constexpr (OP != OP_ICALC)
        bad_bits = mask_bits<E>(a.mask, [&](int e) { return det_row<N, E, NF>(t, e) * N + c; });
    if (a.bg != nullptr) {
#pragma unroll
        for (int e = 0; e < E; ++e) i0[e] += a.bg[det_row<N, E, NF>(t, e) * N + c];
    }
    double acc0 = 0.0, acc1 = 0.0;
#pragma unroll
    for (int e = 0; e < E; ++e) {
        const int q = det_row<N, E, NF>(t, e);
        const float inten = i0[e];
        if constexpr (OP == OP_ICALC) {
            if (active) a.icalc[((size_t)j * N + q) * N + c] = inten;
        } else {
            if (((bad_bits >> e) & 1u) || !active) continue;
            const float iob = iobv[e];
            const float ifl = fmaxf(inten, a.eps);
            if constexpr (OP == OP_LLK) {
                acc0 += (double)llk_model_term(a.llk_model, ifl, iob);
            } else {
                const float d1 = 1.0f - iob / ifl;
                const float d2 = (iob / ifl) / ifl;
                const float j1 = i1[e] * nrm, j2 = i2[e] * nrm;
                acc0 += (double)(d1 * j1);
                acc1 += (double)(d2 * j1 * j1 + 2.0f * d1 * j2);
            }
        }
    }
    if constexpr (OP == OP_LLK) {
        const double r = block_sum(acc0);
        if (threadIdx.x == 0) a.red[blk] = r;
    } else if constexpr (OP == OP_LS || OP == OP_LS2) {
        const double r0 = block_sum(acc0);
        const double r1 = block_sum(acc1);
        if (threadIdx.x == 0) {
            a.red[2 * blk] = r0;
            a.red[2 * blk + 1] = r1;
        }
    }
}

// Plain batched FFT along rows / columns (standalone 2D transform).  Both
// passes remap their blocks so that each XCD takes a contiguous range: the
// column blocks that share 128-byte row lines (and neighbouring rows) are then
// served by one L2 (2048-point frames: 3.9 -> 5.0 TB/s).
template <int N, int DIR>
__global__ __launch_bounds__(256) void k_fft_rows(float2 *data, long rows) {
    using G = RowGeom<N>;
    constexpr int E = G::E, T = G::T, RB = G::RB;
    __shared__ float2 lds[G::LDS_F2];
    const int tid = threadIdx.x, rr = tid / T, t = tid % T;
    const long g = (long)xcd_block(blockIdx.x, gridDim.x) * RB + rr;
    const bool active = g < rows;
    float2 *row = data + (size_t)(active ? g : rows - 1) * N;
    RowLds<N> L(lds, rr);
    float2 u[E];
#pragma unroll
    for (int e = 0; e < E; ++e) u[e] = row[in_index<N, E, DIR>(t, e)];
    fft1d<N, E, DIR>(u, t, L);
    if (active) {
#pragma unroll
        for (int e = 0; e < E; ++e) row[out_index<N, E, DIR>(t, e)] = u[e];
    }
}

// Geometry of the standalone column transform, which reads row-major frames:
// from 128 points up a block takes 16 adjacent columns (128-byte row
// segments; 8 at 2048 points), with 16 elements per thread from 1024 points
// so that the block stays within 1024 threads.
template <int N>
struct FftColGeom {
    static constexpr int E = (N >= 1024) ? 16 : col_e(N), T = N / E;
    static constexpr int CB = (N >= 2048) ? 8 : (N >= 128) ? 16 : col_cb(N);
    static constexpr int THREADS = CB * T;
    static constexpr int LDS_F2 = (FftCfg<N, E>::P > 1) ? N * CB : 1;
    static_assert(THREADS <= 1024, "one block");
};

template <int N, int DIR>
__global__ __launch_bounds__(FftColGeom<N>::THREADS) void k_fft_cols(float2 *data, long count, float scale) {
    using G = FftColGeom<N>;
    constexpr int E = G::E, CB = G::CB;
    extern __shared__ float2 lds_dyn[];
    const int tid = threadIdx.x, cl = tid % CB, t = tid / CB;
    const long g = (long)xcd_block(blockIdx.x, gridDim.x) * CB + cl;
    const bool active = g < count * N;
    const long gg = active ? g : count * N - 1;
    const long f = gg / N;
    const int c = (int)(gg % N);
    float2 *col = data + (size_t)f * N * N + c;
    ColLds<N, CB> L(lds_dyn, cl);
    float2 u[E];
#pragma unroll
    for (int e = 0; e < E; ++e) u[e] = col[(size_t)in_index<N, E, DIR>(t, e) * N];
    fft1d<N, E, DIR>(u, t, L);
    if (active) {
#pragma unroll
        for (int e = 0; e < E; ++e) col[(size_t)out_index<N, E, DIR>(t, e) * N] = cscale(u[e], scale);
    }
}


}  // namespace ptycho
