// passes.hpp - the frame-size specific host passes: launches of the stack
// kernels for frame size N over all stacks of a plan.  Included by exactly
// one translation unit per N (inst_N.hip), which defines the NPass table of
// that size with PTYCHO_DEFINE_PASSES(N).
#pragma once

#include "plan.hpp"
#include "stack_kernels.hpp"
#include "frame_kernels.hpp"

namespace ptycho {

// Kernels whose dynamic LDS exceeds 64 KiB must opt in once per process.
template <class KernelT>
static hipError_t set_dyn_lds(KernelT kern, size_t bytes) {
    if (bytes <= 64 * 1024) return hipSuccess;
    return hipFuncSetAttribute((const void *)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes);
}

template <int N>
static int rows_blocks(int sn) {
    return (int)(((long)sn * N + RowGeom<N>::RB - 1) / RowGeom<N>::RB);
}
template <int N, class G>
static int cols_blocks(int sn) {
    return (int)(((long)sn * N + G::CB - 1) / G::CB);
}

template <int N, int K, int OP, bool NF>
static void launch_cols_joint(const StackArgs &a, hipStream_t s) {
    using G = typename ColJoint<N, K>::G;
    const size_t lds = sizeof(float2) * G::LDS_F2 * ColJoint<N, K>::BUFS;
    static const hipError_t attr = set_dyn_lds(k_cols_joint<N, K, OP, NF>, lds);
    (void)attr;
    const dim3 grid(cols_blocks<N, G>(a.S)), block(G::THREADS);
    hipLaunchKernelGGL((k_cols_joint<N, K, OP, NF>), grid, block, lds, s, a);
}
template <int N, int OP, bool NF>
static void launch_cols_seq(const StackArgs &a, hipStream_t s) {
    using G = typename ColSeqBufs<N, OP>::G;
    const size_t lds = sizeof(float2) * G::LDS_F2 * ColSeqBufs<N, OP>::value;
    static const hipError_t attr = set_dyn_lds(k_cols_seq<N, OP, NF>, lds);
    (void)attr;
    const dim3 grid(cols_blocks<N, G>(a.S)), block(G::THREADS);
    hipLaunchKernelGGL((k_cols_seq<N, OP, NF>), grid, block, lds, s, a);
}

// Forward row pass of input form MODE: the sub-pixel-window instance when the
// plan's windows interpolate, the integer one otherwise.
template <int N, int MODE, bool NF>
static void launch_rows_fwd(StackArgs a, dim3 grid, hipStream_t s) {
    a.side = side_frames<N, MODE, NF>(a.S, a.K);
    if (a.frac != nullptr) hipLaunchKernelGGL((k_rows_fwd<N, MODE, NF, true>), grid, dim3(256), 0, s, a);
    else hipLaunchKernelGGL((k_rows_fwd<N, MODE, NF, false>), grid, dim3(256), 0, s, a);
}

template <int N, int K, int MODE, bool NF>
static void launch_rows_inv(const StackArgs &a, bool wq, hipStream_t s) {
    const dim3 grid((unsigned)(((long)a.S * N + InvRowGeom<N>::RQ - 1) / InvRowGeom<N>::RQ));
    const dim3 block(InvRowGeom<N>::TPM * K);
    // only the DM epilogue reads the view
    if (MODE == OUT_DM && a.frac != nullptr) {
        if (wq) hipLaunchKernelGGL((k_rows_inv<N, K, MODE, true, NF, MODE == OUT_DM>), grid, block, 0, s, a);
        else hipLaunchKernelGGL((k_rows_inv<N, K, MODE, false, NF, MODE == OUT_DM>), grid, block, 0, s, a);
        return;
    }
    if (wq) hipLaunchKernelGGL((k_rows_inv<N, K, MODE, true, NF, false>), grid, block, 0, s, a);
    else hipLaunchKernelGGL((k_rows_inv<N, K, MODE, false, NF, false>), grid, block, 0, s, a);
}

// Small far-field frames: the whole frame in one kernel.
// Sizes of k_frame and k_frame_read: every mode count up to 64 points; at 128
// points the projections of up to two modes (the registers of a 1024-thread
// block hold no more; the line search there needs the kept row transforms).
template <int N, int K>
constexpr bool has_frame() { return N == 32 || N == 64 || (N == 128 && K <= 2); }
template <int N>
constexpr bool has_frame_read() { return N == 32 || N == 64; }

// Whether the plan's projections take a frame per block rather than three
// passes of blocks over all frames.  A block's frame takes a fixed time, so the
// frames of a launch have to fill the chip's 256 CUs by half (DM cycle without
// updates, us, three passes / frame per block: 64^2 x 3 modes 17 / 23 at 64
// frames, 32 / 25 at 200, 216 / 145 at 1500; 128^2 x 1 mode 18 / 29 at 64,
// 50 / 31 at 200, 290 / 183 at 1500; 128^2 x 2 modes 552 / 335 at 1500); one
// mode up to 64 points is as fast or faster at any count (13 / 13 at 8 frames,
// 80 / 43 at 1500).
template <int N, int K>
static bool by_frame(const ptycho_plan_s *p, const float2 *keep) {
    if constexpr (!has_frame<N, K>()) return false;
    if (N == 128 && keep != nullptr) return false;
    return (N <= 64 && K == 1) || p->L.S >= 128;
}

// Whether a read-only pass takes a frame per block.  At 32 points and up to two
// modes at 64 it is the faster way at any count, but for a line search of one
// frame, whose three transforms it does one after the other (32^2 x 1 mode 21
// against 13 us, 64^2 x 4 modes 49 against 20).  At 64 points, three and four
// modes leave room for one block per CU, so the time goes up by a whole round
// with every 256 frames; a round has to be 0.7 full (intensities, 4 modes, us,
// frame per block / three passes: 12 / 9.6 at 16 frames, 12 / 16 at 200, 24 / 21
// at 300, 24 / 26 at 400, 69 / 83 at 1500), and sub-pixel views of two modes
// follow them (10.2 / 9.5 at 32 frames, 11 / 14 at 200).  The likelihood's
// logarithms, which such a block takes with nothing else in flight, turn it from
// the fourth round on (3 modes: 17 / 20 at 200, 42 / 41 at 768, 82 / 75 at 1500).
// Sub-pixel views of four modes at 32 points: 10.5 / 9.6 at 64 frames, 10.6 / 12.5
// at 200.  The line search of four modes spills 100 registers, that of
// sub-pixel views pays for four values a pixel in each of its three transforms:
// they are the faster way only while they save launches, from 3 frames on in
// the first round and in a full second one (4 modes: 50 / 40 us at 2 frames,
// 50 / 77 at 4, 65 / 100 at 256, 112 / 78 at 300, 116 / 120 at 400, 172 / 122 at
// 600, 348 / 266 at 1500).
// Three passes are launched stack by stack, a frame per block all at once, so
// that stacks of fewer frames than a round always take the latter (150 frames
// of 3 modes in stacks of 40: 10 / 37 us).
template <int N, int K, int OP, bool SUB>
static bool read_by_frame(int J, int S) {
    if (S < J && S < 256) return true;
    const int rounds = (J + 255) / 256;
    const bool full = 10L * J >= 7L * 256 * rounds;
    if (OP == OP_LS) {
        if (J == 1) return false;
        if (N == 64 && (K == 4 || (SUB && K >= 2)))
            return rounds == 1 ? (K < 4 || J > 2) : rounds == 2 && full;
        return true;
    }
    if (N == 32) return !(SUB && K == 4) || J > 128;
    return K <= (SUB ? 1 : 2) || (full && (OP != OP_LLK || K == 2 || rounds <= 3));
}

template <int N, int K>
static dim3 frame_blocks(int sn) {
    return dim3((unsigned)((sn + FrameGeom<N, K>::FPB - 1) / FrameGeom<N, K>::FPB));
}
template <int N, int K, int OP, bool SUB>
static void launch_frame_sub(const StackArgs &a, hipStream_t s) {
    const size_t lds = sizeof(float2) * FrameGeom<N, K>::LDS_F2;
    static const hipError_t attr = set_dyn_lds(k_frame<N, K, OP, SUB>, lds);
    (void)attr;
    const dim3 grid = frame_blocks<N, K>(a.S), block(FrameGeom<N, K>::THREADS);
    hipLaunchKernelGGL((k_frame<N, K, OP, SUB>), grid, block, lds, s, a);
}
template <int N, int K, int OP>
static void launch_frame(const StackArgs &a, hipStream_t s) {
    if (a.frac != nullptr) launch_frame_sub<N, K, OP, true>(a, s);
    else launch_frame_sub<N, K, OP, false>(a, s);
}
template <int N, int K, int OP, bool SUB>
static void launch_frame_read(const StackArgs &a, hipStream_t s) {
    const size_t lds = sizeof(float2) * FrameGeom<N, K>::LDS_F2;
    static const hipError_t attr = set_dyn_lds(k_frame_read<N, K, OP, SUB>, lds);
    (void)attr;
    const dim3 grid = frame_blocks<N, K>(a.S), block(FrameGeom<N, K>::THREADS);
    hipLaunchKernelGGL((k_frame_read<N, K, OP, SUB>), grid, block, lds, s, a);
}

// Whether the gradient's inverse rows take the probe sums (k_rows_inv_grad),
// from 128 points on, where a block's rows belong to one frame: integer
// windows only, whose view the kernel reads, and not where position shifts
// need the gradient waves in the scratch.
static bool grad_rows(const ptycho_plan_s *p, const StackArgs &a) {
    return a.frac == nullptr && !p->shifts_in_grad;
}
template <int N, int K, bool NF>
static void launch_rows_inv_grad(ptycho_plan_s *p, const StackArgs &a, int chunks, hipStream_t s) {
    const int blocks = std::max(1, std::min(p->L.gblocks, chunks));
    const dim3 grid((unsigned)(N / InvRowGeom<N>::RQ * blocks)), block(InvRowGeom<N>::TPM * K);
    hipLaunchKernelGGL((k_rows_inv_grad<N, K, NF>), grid, block, 0, s, a, blocks, chunks, p->pnum, p->pden);
}

// One pass over all stacks: forward rows, column op, inverse rows and the
// per-stack gathers.  kind: 0 = AP projection, 1 = DM, 2 = ML gradient.
// Exit waves go to `psi` (all frames) when it is given, else stay in the
// stack scratch.  acc selects the sums taken per stack: the object sums
// (from the inverse row pass's per-frame terms), the probe sums (only for
// the gradient, whose two sums are taken at the same point; by the inverse
// row pass itself or from the exit waves in the scratch).
template <int N, int K, bool NF>
static int project_pass_nk(ptycho_plan_s *p, const float *obj, const float *probe, float *psi, int kind,
                           unsigned acc, bool upd_bg, float2 *keep) {
    const int J = p->d.n_frames, S = p->L.S;
    hipStream_t s = p->stream;
    const bool store = (psi != nullptr);
    const bool wq = (acc & ACC_OBJ) != 0;
    if (wq) {
        Timed tm(p, TC_OTHER);
        const int st = need_probe_intensity(p, probe);
        if (st) return st;
    }
    for (int sidx = 0; sidx < p->L.nstacks; ++sidx) {
        const int s0 = sidx * S, sn = std::min(S, J - s0);
        StackArgs a = stack_args(p, s0, sn, obj, probe);
        a.psi = (const float2 *)psi;
        a.psi_out = (float2 *)psi;
        a.red = p->red + p->red_n;
        if (upd_bg) a.s2 = p->s2;
        if (keep) a.fwd = keep + (size_t)s0 * K * N * N;
        a.colin = a.fwd;
        const bool whole = !NF && by_frame<N, K>(p, keep);
        bool probe_done = false;
        const int chunks = std::max(1, std::min(p->L.gchunks, sn));
        if (whole) {
            if constexpr (has_frame<N, K>() && !NF) {
                if (!wq) a.qbuf = nullptr;
                if (kind == 2) p->red_n += frame_blocks<N, K>(sn).x;
                // one kernel for the three passes: its time counts as the last one's
                { Timed tm(p, TC_ROWS_FWD); }
                { Timed tm(p, TC_COLS); }
                Timed tm(p, TC_ROWS_INV);
                if (kind == 2) launch_frame<N, K, OP_GRAD>(a, s);
                else if (kind == 1) launch_frame<N, K, OP_CORR>(a, s);
                else launch_frame<N, K, OP_PROJECT>(a, s);
            }
        } else {
            if (kind == 2) p->red_n += cols_blocks<N, typename ColJoint<N, K>::G>(sn);
            const dim3 rg(rows_blocks<N>(sn), p->d.n_modes);
            {
                Timed tm(p, TC_ROWS_FWD);
                if (kind == 1) launch_rows_fwd<N, IN_DM, NF>(a, rg, s);
                else launch_rows_fwd<N, IN_PHI, NF>(a, rg, s);
            }
            {
                Timed tm(p, TC_COLS);
                if (kind == 2) launch_cols_joint<N, K, OP_GRAD, NF>(a, s);
                else if (kind == 1) launch_cols_joint<N, K, OP_CORR, NF>(a, s);
                else launch_cols_joint<N, K, OP_PROJECT, NF>(a, s);
            }
            {
                Timed tm(p, TC_ROWS_INV);
                if constexpr (N >= 128) probe_done = kind == 2 && grad_rows(p, a);
                if (probe_done) {
                    if constexpr (N >= 128) launch_rows_inv_grad<N, K, NF>(p, a, chunks, s);
                } else if (kind == 1) launch_rows_inv<N, K, OUT_DM, NF>(a, wq, s);
                else if (store) launch_rows_inv<N, K, OUT_STORE, NF>(a, wq, s);
                else if (acc & ACC_PROBE) launch_rows_inv<N, K, OUT_SCR, NF>(a, wq, s);
                else launch_rows_inv<N, K, OUT_NONE, NF>(a, wq, s);
            }
        }
        if (upd_bg) {
            Timed tm(p, TC_OTHER);
            const int st = launch_bg_accum(p, sn, sidx == 0 ? 1 : 0);
            if (st) return st;
        }
        LAUNCHCHK();
        int st = PTYCHO_OK;
        // ML position shifts from the gradient wave left in the scratch
        if (kind == 2 && p->shifts_in_grad) st = launch_ml_shifts(p, obj, probe, s0, sn);
        if (!st && (acc & ACC_OBJ)) st = object_sums(p, sidx);
        if (!st && probe_done) {
            Timed tm(p, TC_GATHER_PROBE);
            st = reduce_probe(p, chunks, sidx > 0);
        } else if (!st && (acc & ACC_PROBE)) st = probe_sums(p, obj, p->scr, s0, sn, true, sidx > 0);
        if (st) return st;
    }
    return PTYCHO_OK;
}

template <int N>
static int project_pass_n(ptycho_plan_s *p, const float *obj, const float *probe, float *psi, int kind,
                          unsigned acc, bool upd_bg, float2 *keep) {
    return with_k(p->d.n_modes, [&](auto kk) {
        return with_nf(p, [&](auto nf) {
            return project_pass_nk<N, decltype(kk)::value, decltype(nf)::value>(p, obj, probe, psi, kind, acc,
                                                                                  upd_bg, keep);
        });
    });
}

// Read-only forward passes: LLK, icalc, line search.
template <int N, int OP, bool NF>
static int forward_pass_op(ptycho_plan_s *p, const float *obj, const float *probe, const float *dobj,
                           const float *dprobe, float *icalc, int llk_model, const float2 *keep) {
    const bool ls = (OP == OP_LS || OP == OP_LS2);
    const Layout &Lp = p->L;
    const int J = p->d.n_frames;
    const int S = (OP == OP_LS2) ? Lp.S_ls2 : ls ? Lp.S_ls : Lp.S;
    const int nst = (OP == OP_LS2) ? Lp.nstacks_ls2 : ls ? Lp.nstacks_ls : Lp.nstacks;
    hipStream_t s = p->stream;
    for (int sidx = 0; sidx < nst; ++sidx) {
        const int s0 = sidx * S, sn = std::min(S, J - s0);
        StackArgs a = stack_args(p, s0, sn, obj, probe);
        a.dobj = (const float2 *)dobj;
        a.dprobe = (const float2 *)dprobe;
        a.icalc = icalc;
        a.llk_model = llk_model;
        a.red = p->red + p->red_n * (ls ? 2 : 1);
        p->red_n += cols_blocks<N, typename ColSeqBufs<N, OP>::G>(sn);
        if (OP == OP_LS2) a.colin = keep + (size_t)s0 * p->d.n_modes * N * N;
        const dim3 rg(rows_blocks<N>(sn), p->d.n_modes);
        {
            Timed tm(p, TC_ROWS_FWD);
            if (OP == OP_LS2) launch_rows_fwd<N, IN_LS2, NF>(a, rg, s);
            else if (ls) launch_rows_fwd<N, IN_LS, NF>(a, rg, s);
            else launch_rows_fwd<N, IN_PHI, NF>(a, rg, s);
        }
        {
            Timed tm(p, TC_COLS);
            launch_cols_seq<N, OP, NF>(a, s);
        }
        LAUNCHCHK();
    }
    return PTYCHO_OK;
}

// The same on small far-field frames: one launch over all frames (a block per
// frame, no scratch).
template <int N, int OP>
static int frame_pass_op(ptycho_plan_s *p, const float *obj, const float *probe, const float *dobj,
                         const float *dprobe, float *icalc, int llk_model) {
    StackArgs a = stack_args(p, 0, p->d.n_frames, obj, probe);
    a.dobj = (const float2 *)dobj;
    a.dprobe = (const float2 *)dprobe;
    a.icalc = icalc;
    a.llk_model = llk_model;
    a.red = p->red;
    { Timed tm(p, TC_ROWS_FWD); }
    Timed tm(p, TC_COLS);
    return with_k(p->d.n_modes, [&](auto kk) {
        constexpr int K = decltype(kk)::value;
        p->red_n = frame_blocks<N, K>(a.S).x;
        if (a.frac != nullptr) launch_frame_read<N, K, OP, true>(a, p->stream);
        else launch_frame_read<N, K, OP, false>(a, p->stream);
        LAUNCHCHK();
        return (int)PTYCHO_OK;
    });
}

template <int N>
static int forward_pass_n(ptycho_plan_s *p, int op, const float *obj, const float *probe, const float *dobj,
                          const float *dprobe, float *icalc, int llk_model, const float2 *keep) {
    return with_nf(p, [&](auto nf) {
        constexpr bool NF = decltype(nf)::value;
        if constexpr (has_frame_read<N>() && !NF) {
            // the gradient pass of a plan whose projections take a frame per block
            // kept no row transforms
            if (op == OP_LS2 &&
                with_k(p->d.n_modes, [&](auto kk) { return (int)by_frame<N, decltype(kk)::value>(p, keep); }))
                op = OP_LS;
            const auto whole = [&](auto o) {
                constexpr int OP = decltype(o)::value;
                const int J = p->d.n_frames, S = p->L.S;
                return with_k(p->d.n_modes, [&](auto kk) {
                    constexpr int K = decltype(kk)::value;
                    return (int)(p->pos_ready ? read_by_frame<N, K, OP, true>(J, S)
                                              : read_by_frame<N, K, OP, false>(J, S));
                }) != 0;
            };
            if (op == OP_LLK && whole(std::integral_constant<int, OP_LLK>()))
                return frame_pass_op<N, OP_LLK>(p, obj, probe, dobj, dprobe, icalc, llk_model);
            if (op == OP_ICALC && whole(std::integral_constant<int, OP_ICALC>()))
                return frame_pass_op<N, OP_ICALC>(p, obj, probe, dobj, dprobe, icalc, llk_model);
            if (op == OP_LS && whole(std::integral_constant<int, OP_LS>()))
                return frame_pass_op<N, OP_LS>(p, obj, probe, dobj, dprobe, icalc, llk_model);
        }
        switch (op) {
            case OP_LLK: return forward_pass_op<N, OP_LLK, NF>(p, obj, probe, dobj, dprobe, icalc, llk_model, keep);
            case OP_ICALC: return forward_pass_op<N, OP_ICALC, NF>(p, obj, probe, dobj, dprobe, icalc, llk_model, keep);
            case OP_LS: return forward_pass_op<N, OP_LS, NF>(p, obj, probe, dobj, dprobe, icalc, llk_model, keep);
            case OP_LS2: return forward_pass_op<N, OP_LS2, NF>(p, obj, probe, dobj, dprobe, icalc, llk_model, keep);
            default: return fail(PTYCHO_E_INVALID, "internal: unknown forward op");
        }
    });
}

template <int N>
static int fft2_n(int32_t count, float *data, int32_t dir, hipStream_t s) {
    const long rows = (long)count * N;
    const int rb = (int)((rows + RowGeom<N>::RB - 1) / RowGeom<N>::RB);
    using FG = FftColGeom<N>;
    const int cbk = (int)((rows + FG::CB - 1) / FG::CB);
    const size_t lds = sizeof(float2) * FG::LDS_F2;
    const float scale = 1.0f / (float)N;
    if (dir < 0) {
        static const hipError_t attr = set_dyn_lds(k_fft_cols<N, -1>, lds);
        (void)attr;
        hipLaunchKernelGGL((k_fft_rows<N, -1>), dim3(rb), dim3(256), 0, s, (float2 *)data, rows);
        hipLaunchKernelGGL((k_fft_cols<N, -1>), dim3(cbk), dim3(FG::THREADS), lds, s, (float2 *)data,
                           (long)count, scale);
    } else {
        static const hipError_t attr = set_dyn_lds(k_fft_cols<N, 1>, lds);
        (void)attr;
        hipLaunchKernelGGL((k_fft_rows<N, 1>), dim3(rb), dim3(256), 0, s, (float2 *)data, rows);
        hipLaunchKernelGGL((k_fft_cols<N, 1>), dim3(cbk), dim3(FG::THREADS), lds, s, (float2 *)data,
                           (long)count, scale);
    }
    LAUNCHCHK();
    return PTYCHO_OK;
}

static hipError_t set_twiddles_here(const float2 *host) {
    return hipMemcpyToSymbol(HIP_SYMBOL(g_twiddle), host, sizeof(float2) * TW_MAX);
}

}  // namespace ptycho

// The table is built inside a host function, so that the device compilation
// emits no host data but still instantiates the kernels the passes launch.
#define PTYCHO_DEFINE_PASSES(NN)                                                                       \
    namespace ptycho {                                                                                \
    const NPass *passes_##NN() {                                                                      \
        static const NPass t = {NN, project_pass_n<NN>, forward_pass_n<NN>, fft2_n<NN>, set_twiddles_here}; \
        return &t;                                                                                    \
    }                                                                                                 \
    }
