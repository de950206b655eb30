// frame_kernels.hpp - the stack passes of small far-field frames (32, 64 and
// 128 points): one kernel takes a frame from the object view to its new exit
// waves, both transforms of the 2D FFT in registers and LDS.
//
// A frame-mode plane of N x N complex values fits the LDS of one CU up to 128
// points (128 KiB), so the stack scratch between the row and the column passes
// is not needed: a projection reads the old exit waves and writes the new ones
// and q, and the line search reads nothing but the object and the probe.  The
// plane is the exchange buffer of the transforms; a thread holds 16 values.
//
// The y transform comes first: its threads own columns, so that every access
// to row-major data (views, probe, exit waves, q) covers whole rows; the x
// transform's exchanges stay within one wavefront (the N / 16 threads of a row
// are neighbouring lanes) and need no block barrier.
//
// Up to 64 points a block holds the planes of all K modes and gives each mode
// its own wavefronts, which meet twice: to sum the intensity and to sum q.
// At 128 points one plane fills the LDS, and the modes are transformed one
// after the other by the same threads, all kept in registers.
#pragma once

#include "common.hpp"

namespace ptycho {

template <int N, int K>
struct FrameGeom {
    static constexpr int E = 16, T = N / E;             // values and threads per transform
    static constexpr int TPF = N * T;                   // threads per plane (whole wavefronts)
    static constexpr int KG = N <= 64 ? K : 1;          // modes side by side in a block
    static constexpr int KS = K / KG;                   // modes one after the other
    // frames per block: about 256 threads, at least two frames at 32 points
    // (the reduction partials hold one value per two frames there)
    static constexpr int FPB0 = KG * TPF >= 256 ? 1 : 256 / (KG * TPF);
    static constexpr int FPB = N == 32 && FPB0 < 2 ? 2 : FPB0;
    static constexpr int THREADS = TPF * KG * FPB;
    static constexpr int LDS_F2 = FPB * KG * N * N;
};

// Exchange of the 5 low bits of a slot by bits of x and y, so that the 32
// lanes of an LDS cycle hit distinct 8-byte slots in every access of the x
// passes (lanes: T threads x 32 / T rows; strides 1, 4, 8 and 16 in x).  The y
// passes touch whole rows and are free of conflicts under any such exchange.
// Both are linear over XOR: the swizzle of an index whose bits come from two
// parts is the XOR of the parts' swizzles.
template <int N>
__device__ __forceinline__ constexpr int swz_x(int x) {
    return N == 128 ? ((x & 32) >> 3) ^ ((x & 64) >> 6) : 0;
}
template <int N>
__device__ __forceinline__ constexpr int swz_y(int y) {
    return N == 128  ? ((y & 1) * 9) ^ ((y & 2) * 9)
           : N == 64 ? ((y & 1) * 4) ^ ((y & 2) * 5) ^ (((y & 4) >> 2) * 17)
                     : ((y & 1) * 2) ^ ((y & 2) * 8) ^ (((y & 4) >> 2) * 5) ^ (((y & 8) >> 3) * 9);
}

typedef __attribute__((address_space(3))) char lds_char;
typedef __attribute__((address_space(3))) float2 lds_float2;

// The transform along y in column c, or along x in row r.  An index is a part
// known at run time and one known at compile time without bits in common; the
// compile-time part becomes one XOR of the low slot bits and the offset of the
// LDS instruction.  The plane is 256-byte aligned.
template <int N>
struct PlaneCol {
    lds_char *p;
    int c;
    __device__ __forceinline__ lds_float2 *at(int i, int k) const {
        const int b = ((i * N + c) ^ swz_x<N>(c) ^ swz_y<N>(i)) * 8;
        return (lds_float2 *)(p + (b ^ (swz_y<N>(k) * 8)) + k * N * 8);
    }
    __device__ __forceinline__ float2 ld(int i, int k) const {
        lds_float2 *q = at(i, k);
        return make_float2(q->x, q->y);
    }
    __device__ __forceinline__ void st(int i, int k, float2 v) {
        lds_float2 *q = at(i, k);
        q->x = v.x;
        q->y = v.y;
    }
    __device__ __forceinline__ void sync() const { __syncthreads(); }
};
template <int N>
struct PlaneRow {                    // the lanes of one wavefront hold whole rows
    lds_char *p;
    int r;
    __device__ __forceinline__ lds_float2 *at(int i, int k) const {
        const int b = ((r * N + i) ^ swz_y<N>(r) ^ swz_x<N>(i)) * 8;
        return (lds_float2 *)(p + (b ^ ((k ^ swz_x<N>(k)) * 8)));
    }
    __device__ __forceinline__ float2 ld(int i, int k) const {
        lds_float2 *q = at(i, k);
        return make_float2(q->x, q->y);
    }
    __device__ __forceinline__ void st(int i, int k, float2 v) {
        lds_float2 *q = at(i, k);
        q->x = v.x;
        q->y = v.y;
    }
    __device__ __forceinline__ void sync() const {
        // one wavefront's LDS accesses complete in order; keep the compiler's order too
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
    }
};

// The y phase's transform thread t: the same for all lanes of a wavefront from
// 64 points on (a wavefront then owns 64 columns of a row), so it lives in a
// scalar register and the row addresses of the y phase are scalar too.  Each
// transform takes an opaque copy of its thread index: the twiddles and
// addresses of one transform are then not kept in registers for the next.
template <int N>
__device__ __forceinline__ int opaque_t(int t) {
    if constexpr (N >= 64) {
        asm volatile("" : "+s"(t));
        return t;
    } else {
        return opaque(t);
    }
}

// Forward 2D transform: u holds column c (values y = in_index(t, e)) on entry
// and row r (values x = out_index(tr, e)) on return.
template <int N>
__device__ __forceinline__ void frame_forward(float2 *u, PlaneCol<N> C, int t, PlaneRow<N> R, int tr) {
    constexpr int E = 16, RI = FirstRadix<N, E, -1>::value, RO = LastRadix<N, E, -1>::value;
    t = opaque_t<N>(t);
    tr = opaque(tr);
    C.c = opaque(C.c);
    R.r = opaque(R.r);
    fft1d<N, E, -1>(u, t, C);
    C.sync();
#pragma unroll
    for (int e = 0; e < E; ++e) C.st(t, elem_const<N, E, RO>(e), u[e]);
    C.sync();
#pragma unroll
    for (int e = 0; e < E; ++e) u[e] = R.ld(tr, elem_const<N, E, RI>(e));
    fft1d<N, E, -1>(u, tr, R);
}
// The inverse, from rows back to columns (y = out_index<+1>(t, e)).
template <int N>
__device__ __forceinline__ void frame_inverse(float2 *u, PlaneCol<N> C, int t, PlaneRow<N> R, int tr) {
    constexpr int E = 16, RI = FirstRadix<N, E, +1>::value, RO = LastRadix<N, E, +1>::value;
    t = opaque_t<N>(t);
    tr = opaque(tr);
    C.c = opaque(C.c);
    R.r = opaque(R.r);
    C.sync();                        // every wavefront is done with the plane's columns
    fft1d<N, E, +1>(u, tr, R);
    R.sync();
#pragma unroll
    for (int e = 0; e < E; ++e) R.st(tr, elem_const<N, E, RO>(e), u[e]);
    C.sync();
#pragma unroll
    for (int e = 0; e < E; ++e) u[e] = C.ld(t, elem_const<N, E, RI>(e));
    fft1d<N, E, +1>(u, t, C);
}

// A thread's place: frame slot s (frame j), mode k of those side by side,
// column c with transform thread t (y phase), row r with thread tr (x phase).
template <int N, int K>
struct FrameThread {
    using G = FrameGeom<N, K>;
    int blk, f, k, s, j, i, c, t, r, tr;
    bool active;
    int2 o;
    __device__ __forceinline__ FrameThread(const StackArgs &a) {
        // a wavefront works on one plane
        const int w = G::THREADS == G::TPF ? 0 : __builtin_amdgcn_readfirstlane(threadIdx.x / G::TPF);
        f = w / G::KG;
        k = w % G::KG;
        i = G::THREADS == G::TPF ? (int)threadIdx.x : (int)threadIdx.x % G::TPF;
        blk = xcd_block(blockIdx.x, gridDim.x);
        const int slot = blk * G::FPB + f;
        active = slot < a.S;
        s = active ? slot : a.S - 1;
        j = a.order[a.s0 + s];
        o = a.offs[j];
        c = i % N;
        t = N >= 64 ? __builtin_amdgcn_readfirstlane(i / N) : i / N;
        r = i / G::T;
        tr = i % G::T;
    }
};

// Sub-pixel views read four object values per pixel: their loads are issued
// for four pixels at a time, not all at once, which would spill.
template <bool SUB>
__device__ __forceinline__ void view_fence(int e) {
    if constexpr (SUB)
        if (e % 4 == 3) __builtin_amdgcn_sched_barrier(0);
}

// The object view (or that of a direction) at pixel (y, c) of the frame.
template <bool SUB>
__device__ __forceinline__ float2 frame_view(const StackArgs &a, const float2 *b, int2 o, float2 fr, int y, int c) {
    if constexpr (SUB) {
        return view_at(b, view_row(a.Ny, a.Nx, o, fr, y), c);
    } else {
        const float2 *row = b + ((size_t)(o.x + y) * a.Nx + o.y);
        return row[(unsigned)c];
    }
}

// One frame: exit waves (IN_PHI) or 2 Phi - Psi (OP_CORR), the Fourier step,
// and back.  At 128 points with two modes the kernel sits at the 128 registers
// that a 1024-thread block may hold and spills 41 to 55 more, a seventh of its
// time (500 frames, AP: 109 us, 90 with butterflies that need 20 registers less
// and round worse).  New exit waves go to psi_out when it is given (AP, DM) or to the
// stack scratch (OP_GRAD); q = sum_k conj(P_k) Psi_k to qbuf when it is given.
template <int N, int K, int OP, bool SUB>
__global__ __launch_bounds__((FrameGeom<N, K>::THREADS)) void k_frame(StackArgs a) {
    using G = FrameGeom<N, K>;
    constexpr int E = G::E, KS = G::KS, KG = G::KG;
    constexpr bool DM = OP == OP_CORR;
    constexpr float nrm = 1.0f / ((float)N * (float)N);
    // Where the planes leave room for one block per CU, nothing hides a load that
    // waits behind a transform: the observed data, the probe and the DM form's
    // view are loaded before it (64 x 64, DM, three modes: 333 frames 55 -> 52 us,
    // 1500 frames 163 -> 161; four modes 69 -> 65, 204 -> 200).  At 128 points
    // and one mode, 16 waves of up to 115 registers, it gave nothing (2000
    // frames: 288 -> 292 us DM, 218 -> 227 AP).
    constexpr bool AHEAD = N == 64 && G::LDS_F2 * sizeof(float2) > 80 * 1024;
    constexpr bool AHEAD_OBJ = AHEAD && DM && !SUB;
    extern __shared__ __attribute__((aligned(1024))) float2 lds_frame[];
    const FrameThread<N, K> th(a);
    float2 *plane = lds_frame + (th.f * KG + th.k) * N * N;
    PlaneCol<N> C{(lds_char *)plane, th.c};
    PlaneRow<N> R{(lds_char *)plane, th.r};
    const size_t n2 = (size_t)N * N;
    const float2 fr = SUB ? a.frac[th.j] : make_float2(0.0f, 0.0f);

    auto form = [&](float2 *u, int k) {
        const int t = opaque_t<N>(th.t);
        const unsigned c = opaque(th.c);
        const float2 *p = a.probe + k * n2;
        const float2 *ps = a.psi + ((size_t)th.j * K + k) * n2;
#pragma unroll
        for (int e = 0; e < E; ++e) {
            const int y = in_index<N, E, -1>(t, e);
            const float2 phi = cmul(frame_view<SUB>(a, a.obj, th.o, fr, y, c), (p + y * N)[c]);
            if constexpr (DM) {
                const float2 v = ld_stream(ps + y * N + c);
                u[e] = make_float2(2.0f * phi.x - v.x, 2.0f * phi.y - v.y);
            } else {
                u[e] = phi;
            }
            view_fence<SUB>(e);
        }
    };

    // the data of the pixels (r, x) this thread owns
    float iobv[E], sc[E];
    auto pixel = [&](int e) { return (unsigned)(th.r * N + th.tr) + elem_const<N, E, LastRadix<N, E, -1>::value>(e); };
    auto load_iobs = [&] {
        const float *io = a.iobs + (size_t)th.j * n2;
#pragma unroll
        for (int e = 0; e < E; ++e) iobv[e] = io[pixel(e)];
    };
    float2 u[KS][E];
#pragma unroll
    for (int m = 0; m < KS; ++m) {
        form(u[m], th.k + m);
        if constexpr (AHEAD) load_iobs();
        frame_forward<N>(u[m], C, th.t, R, th.tr);
    }
    if constexpr (!AHEAD) load_iobs();
    const unsigned bad_bits = mask_bits<E>(a.mask, pixel);
    // intensity -> scale
#pragma unroll
    for (int e = 0; e < E; ++e) {
        sc[e] = 0.0f;
#pragma unroll
        for (int m = 0; m < KS; ++m) sc[e] += cnorm(u[m][e]);
    }
    if constexpr (KG > 1) {
        // sum over the modes of the block, in mode order, through the planes
        float *own = (float *)plane + th.i;
        const float *all = (const float *)(lds_frame + th.f * KG * N * N) + th.i;
        __syncthreads();
#pragma unroll
        for (int e = 0; e < E; ++e) own[e * G::TPF] = sc[e];
        __syncthreads();
#pragma unroll
        for (int e = 0; e < E; ++e) {
            sc[e] = all[e * G::TPF];
#pragma unroll
            for (int m = 1; m < KG; ++m) sc[e] += all[m * 2 * N * N + e * G::TPF];
        }
    }
    double acc = 0.0;
    {
#pragma unroll
        for (int e = 0; e < E; ++e) sc[e] *= nrm;
        if (a.bg != nullptr) {
#pragma unroll
            for (int e = 0; e < E; ++e) sc[e] += a.bg[pixel(e)];
        }
#pragma unroll
        for (int e = 0; e < E; ++e) {
            const unsigned x = pixel(e);
            const float inten = sc[e];
            const bool bad = (bad_bits >> e) & 1u;
            const float iob = iobv[e];
            if constexpr (OP == OP_PROJECT) {
                const float q = iob / fmaxf(inten, a.eps);
                sc[e] = bad ? nrm : sqrtf(q) * nrm;
                if (a.s2 != nullptr && th.active && th.k == 0) (a.s2 + (size_t)th.s * n2)[x] = bad ? 1.0f : q;
            } else if constexpr (OP == OP_CORR) {
                sc[e] = bad ? 0.0f : (sqrtf(iob / fmaxf(inten, a.eps)) - 1.0f) * nrm;
            } else {
                const float ifl = fmaxf(inten, a.eps);
                sc[e] = bad ? 0.0f : (1.0f - iob / ifl) * nrm;
                if (!bad && th.active && th.k == 0) acc += (double)llk_term(ifl, iob);
            }
        }
    }

    float2 q[E];
#pragma unroll
    for (int m = 0; m < KS; ++m) {
        const int k = th.k + m;
#pragma unroll
        for (int e = 0; e < E; ++e) u[m][e] = cscale(u[m][e], sc[e]);
        const float2 *p = a.probe + k * n2;
        float2 pv[AHEAD ? E : 1], ov[AHEAD_OBJ ? E : 1];
        if constexpr (AHEAD) {
            const int t = opaque_t<N>(th.t);
            const unsigned c = opaque(th.c);
#pragma unroll
            for (int e = 0; e < E; ++e) {
                const int y = out_index<N, E, +1>(t, e);
                pv[e] = (p + y * N)[c];
                if constexpr (AHEAD_OBJ) ov[e] = frame_view<SUB>(a, a.obj, th.o, fr, y, c);
            }
        }
        frame_inverse<N>(u[m], C, th.t, R, th.tr);
        const int t = opaque_t<N>(th.t);
        const unsigned c = opaque(th.c);
        float2 *ps = a.psi_out + ((size_t)th.j * K + k) * n2;
        float2 *scr = a.scr + ((size_t)th.s * K + k) * n2;
#pragma unroll
        for (int e = 0; e < E; ++e) {
            const int y = out_index<N, E, +1>(t, e);
            const float2 pe = AHEAD ? pv[AHEAD ? e : 0] : (p + y * N)[c];
            float2 w = u[m][e];
            if constexpr (AHEAD_OBJ) w = cadd(cmul(ov[e], pe), w);
            else if constexpr (DM) w = cadd(cmul(frame_view<SUB>(a, a.obj, th.o, fr, y, c), pe), w);
            if (th.active) {
                if constexpr (OP == OP_GRAD) scr[scr_at<N>(y, c)] = w;
                else if (a.psi_out != nullptr) st_stream(ps + y * N + c, w);
            }
            const float2 qe = cmulc(pe, w);
            q[e] = m == 0 ? qe : cadd(q[e], qe);
            view_fence<SUB && DM>(e);
        }
    }
    if (a.qbuf != nullptr) {
        if constexpr (KG > 1) {
            float2 *own = plane + th.i;
            const float2 *all = lds_frame + th.f * KG * N * N + th.i;
            __syncthreads();
#pragma unroll
            for (int e = 0; e < E; ++e) own[e * G::TPF] = q[e];
            __syncthreads();
            // mode k's threads sum and write the values e = k, k + K, ...
            float2 *qs = a.qbuf + (size_t)th.s * n2;
#pragma unroll
            for (int e0 = 0; e0 < E; e0 += KG) {
                const int e = e0 + th.k;
                if (e >= E || !th.active) break;
                float2 v = all[e * G::TPF];
#pragma unroll
                for (int m = 1; m < KG; ++m) v = cadd(v, all[m * N * N + e * G::TPF]);
                st_stream(qs + out_index<N, E, +1>(th.t, e) * N + th.c, v);
            }
        } else if (th.active) {
            float2 *qs = a.qbuf + (size_t)th.s * n2;
#pragma unroll
            for (int e = 0; e < E; ++e) st_stream(qs + out_index<N, E, +1>(th.t, e) * N + (unsigned)th.c, q[e]);
        }
    }
    if constexpr (OP == OP_GRAD) {
        const double v = block_sum(acc);
        if (threadIdx.x == 0) a.red[th.blk] = v;
    }
}

// Read-only steps of one frame: LLK, calculated intensity, and the line
// search's two coefficients (A = P O, B = P dO + dP O, C = dP dO of each mode,
// one transform after the other).  The modes are side by side in a block as
// above; their intensities and first- and second-order terms are summed
// through the planes.  The line search keeps three sums and two waves, 112
// values, beside the transform: at 64 points it spills 12 registers with three
// modes (168 of its own) and 103 to 106 with four (128), which is why it then
// takes three passes at most counts (see read_by_frame).
template <int N, int K, int OP, bool SUB>
__global__ __launch_bounds__((FrameGeom<N, K>::THREADS)) void k_frame_read(StackArgs a) {
    using G = FrameGeom<N, K>;
    constexpr int E = G::E, KS = G::KS, KG = G::KG;
    constexpr bool LS = OP == OP_LS;
    constexpr float nrm = 1.0f / ((float)N * (float)N);
    extern __shared__ __attribute__((aligned(1024))) float2 lds_frame[];
    const FrameThread<N, K> th(a);
    float2 *plane = lds_frame + (th.f * KG + th.k) * N * N;
    PlaneCol<N> C{(lds_char *)plane, th.c};
    PlaneRow<N> R{(lds_char *)plane, th.r};
    const size_t n2 = (size_t)N * N;
    const float2 fr = SUB ? a.frac[th.j] : make_float2(0.0f, 0.0f);

    float i0[E], i1[LS ? E : 1], i2[LS ? E : 1];
#pragma unroll
    for (int e = 0; e < E; ++e) {
        i0[e] = 0.0f;
        if constexpr (LS) i1[e] = i2[e] = 0.0f;
    }
#pragma unroll 1
    for (int m = 0; m < KS; ++m) {
        const int k = th.k + m;
        const float2 *p = a.probe + k * n2, *dp = a.dprobe + k * n2;
        float2 A[E];
        {
            const int t = opaque_t<N>(th.t);
            const unsigned c = opaque(th.c);
#pragma unroll
            for (int e = 0; e < E; ++e) {
                const int y = in_index<N, E, -1>(t, e);
                A[e] = cmul(frame_view<SUB>(a, a.obj, th.o, fr, y, c), (p + y * N)[c]);
                view_fence<SUB>(e);
            }
        }
        frame_forward<N>(A, C, th.t, R, th.tr);
#pragma unroll
        for (int e = 0; e < E; ++e) i0[e] += cnorm(A[e]);
        if constexpr (LS) {
#pragma unroll 1
            for (int set = 1; set < 3; ++set) {
                float2 V[E];
                const int t = opaque_t<N>(th.t);
                const unsigned c = opaque(th.c);
#pragma unroll
                for (int e = 0; e < E; ++e) {
                    const int y = in_index<N, E, -1>(t, e);
                    const float2 dv = frame_view<SUB>(a, a.dobj, th.o, fr, y, c), dq = (dp + y * N)[c];
                    V[e] = set == 1 ? cadd(cmul(dv, (p + y * N)[c]), cmul(frame_view<SUB>(a, a.obj, th.o, fr, y, c), dq))
                                    : cmul(dv, dq);
                    view_fence<SUB>(e);
                }
                frame_forward<N>(V, C, th.t, R, th.tr);
#pragma unroll
                for (int e = 0; e < E; ++e) {
                    const float d = 2.0f * cmulc(A[e], V[e]).x;
                    if (set == 1) {
                        i1[e] += d;
                        i2[e] += cnorm(V[e]);
                    } else {
                        i2[e] += d;
                    }
                }
            }
        }
    }
    if constexpr (KG > 1) {
        auto over_modes = [&](float (&v)[E]) {
            float *own = (float *)plane + th.i;
            const float *all = (const float *)(lds_frame + th.f * KG * N * N) + th.i;
            __syncthreads();
#pragma unroll
            for (int e = 0; e < E; ++e) own[e * G::TPF] = v[e];
            __syncthreads();
#pragma unroll
            for (int e = 0; e < E; ++e) {
                v[e] = all[e * G::TPF];
#pragma unroll
                for (int m = 1; m < KG; ++m) v[e] += all[m * 2 * N * N + e * G::TPF];
            }
        };
        over_modes(i0);
        if constexpr (LS) {
            over_modes(i1);
            over_modes(i2);
        }
    }

    const float *io = a.iobs + (size_t)th.j * n2;
    auto pixel = [&](int e) { return (unsigned)(th.r * N + th.tr) + elem_const<N, E, LastRadix<N, E, -1>::value>(e); };
    float iobv[E];
    unsigned bad_bits = 0;
#pragma unroll
    for (int e = 0; e < E; ++e) {
        i0[e] *= nrm;
        if constexpr (OP != OP_ICALC) iobv[e] = io[pixel(e)];
    }
    if constexpr (OP != OP_ICALC) bad_bits = mask_bits<E>(a.mask, pixel);
    if (a.bg != nullptr) {
#pragma unroll
        for (int e = 0; e < E; ++e) i0[e] += a.bg[pixel(e)];
    }
    double acc0 = 0.0, acc1 = 0.0;
#pragma unroll
    for (int e = 0; e < E; ++e) {
        // each mode's threads take the pixels of their elements e = k, k + K, ...
        if (KG > 1 && e % KG != th.k) continue;
        const unsigned x = pixel(e);
        const float inten = i0[e];
        if constexpr (OP == OP_ICALC) {
            if (th.active) (a.icalc + (size_t)th.j * n2)[x] = inten;
        } else {
            if (((bad_bits >> e) & 1u) || !th.active) continue;
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
        const double v = block_sum(acc0);
        if (threadIdx.x == 0) a.red[th.blk] = v;
    } else if constexpr (LS) {
        const double v0 = block_sum(acc0);
        const double v1 = block_sum(acc1);
        if (threadIdx.x == 0) {
            a.red[2 * th.blk] = v0;
            a.red[2 * th.blk + 1] = v1;
        }
    }
}

}  // namespace ptycho
