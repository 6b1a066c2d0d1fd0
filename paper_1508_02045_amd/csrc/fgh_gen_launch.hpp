// fgh_gen_launch.hpp -- launches of the run-time-length passes for one precision.
#pragma once
#include "fgh_dispatch.hpp"
#include "fgh_gen.hpp"

namespace fgh {

// Whether the dense step of a length is summed in two chains: p is no prime.
inline bool split_sums(const Axis& ax) { return ax.rad[ax.nst - 1] != ax.p; }

// NI: 0 (both steps in registers), 2 or 4 dense products per wavefront, plus kGenSplit.
#define FGH_GEN_NI(NI, AX, CALL)                                             \
    switch (NI) {                                                           \
        case 0: return CALL(0);                                             \
        case 1:                                                             \
        case 2: return split_sums(AX) ? CALL(2 + kGenSplit) : CALL(2);      \
        case 3:                                                             \
        case 4: return split_sums(AX) ? CALL(4 + kGenSplit) : CALL(4);      \
    }                                                                       \
    return hipErrorInvalidValue

template <typename T, int D, int NI>
static hipError_t gen_first_ni(const OpPlan& op, const FirstArgs<T>& fa, int opc, unsigned nblk)
{
    LAUNCH_LDS_T((kg_first<T, D, NI>), dim3(nblk), op.th_row, op.lds_first_v2, op.stream, fa, opc);
    return hipGetLastError();
}

template <typename T>
hipError_t gen_first(const OpPlan& op, const FirstArgs<T>& fa, int opc, unsigned nblk)
{
#define C(N) (op.g.d == 2 ? gen_first_ni<T, 2, N>(op, fa, opc, nblk) : gen_first_ni<T, 3, N>(op, fa, opc, nblk))
    FGH_GEN_NI(op.ni_row, fa.ax, C);
#undef C
}

template <typename T, int D, int EPI, int NI>
static hipError_t gen_last_ni(const OpPlan& op, const LastArgs<T>& la, unsigned nblk)
{
    LAUNCH_LDS_T((kg_last<T, D, EPI, NI>), dim3(nblk), op.th_row, op.lds_last_v2, op.stream, la);
    return hipGetLastError();
}

template <typename T, int EPI>
static hipError_t gen_last_epi(const OpPlan& op, const LastArgs<T>& la, unsigned nblk)
{
#define C(N) (op.g.d == 2 ? gen_last_ni<T, 2, EPI, N>(op, la, nblk) : gen_last_ni<T, 3, EPI, N>(op, la, nblk))
    FGH_GEN_NI(op.ni_row, la.ax, C);
#undef C
}

// Single precision has these passes for fgh_apply_f32 alone (plain epilogue, G^ multiplier).
template <typename T>
hipError_t gen_last(const OpPlan& op, const LastArgs<T>& la, int epi, unsigned nblk)
{
    if (epi == EPI_STORE) return gen_last_epi<T, EPI_STORE>(op, la, nblk);
    if constexpr (sizeof(T) == 8) {
        switch (epi) {
            case EPI_RICH: return gen_last_epi<T, EPI_RICH>(op, la, nblk);
            case EPI_CGR: return gen_last_epi<T, EPI_CGR>(op, la, nblk);
            case EPI_CGRX: return gen_last_epi<T, EPI_CGRX>(op, la, nblk);
            case EPI_CHEB: return gen_last_epi<T, EPI_CHEB>(op, la, nblk);
            case EPI_EM: return gen_last_epi<T, EPI_EM>(op, la, nblk);
        }
    }
    return hipErrorInvalidValue;
}

template <typename T, int D, int EPI, int NI>
static hipError_t gen_lastfirst_ni(const OpPlan& op, const LastArgs<T>& la, unsigned nblk)
{
    LAUNCH_LDS_T((kg_lastfirst<T, D, EPI, NI>), dim3(nblk), op.th_row, op.lds_fused, op.stream, la);
    return hipGetLastError();
}

template <typename T, int EPI>
static hipError_t gen_lastfirst_epi(const OpPlan& op, const LastArgs<T>& la, unsigned nblk)
{
#define C(N) (op.g.d == 2 ? gen_lastfirst_ni<T, 2, EPI, N>(op, la, nblk) : gen_lastfirst_ni<T, 3, EPI, N>(op, la, nblk))
    FGH_GEN_NI(op.ni_row, la.ax, C);
#undef C
}

// Double precision only, as the loops.
template <typename T>
hipError_t gen_lastfirst(const OpPlan& op, const LastArgs<T>& la, int epi, unsigned nblk)
{
    if constexpr (sizeof(T) == 8) {
        switch (epi) {
            case EPI_RICH: return gen_lastfirst_epi<T, EPI_RICH>(op, la, nblk);
            case EPI_CHEB: return gen_lastfirst_epi<T, EPI_CHEB>(op, la, nblk);
            case EPI_EM: return gen_lastfirst_epi<T, EPI_EM>(op, la, nblk);
        }
    }
    return hipErrorInvalidValue;
}

template <typename T, int NI>
static hipError_t gen_axis_ni(const OpPlan& op, const AxisArgs<T>& xa, bool inv, int B)
{
    const dim3 grid(axis_blocks(xa));
    if (inv)
        LAUNCH_LDS_T((kg_axis<T, true, NI>), grid, op.th_axis, op.lds_axis, op.stream, xa, B);
    else
        LAUNCH_LDS_T((kg_axis<T, false, NI>), grid, op.th_axis, op.lds_axis, op.stream, xa, B);
    return hipGetLastError();
}

template <typename T>
hipError_t gen_axis(const OpPlan& op, const AxisArgs<T>& xa, bool inv, int B)
{
#define C(N) gen_axis_ni<T, N>(op, xa, inv, B)
    FGH_GEN_NI(op.ni_axis, xa.ax, C);
#undef C
}

template <typename T, int D, int NI>
static hipError_t gen_middle_ni(const OpPlan& op, const MidArgs<T>& ma, int mult)
{
    if (mult == MULT_G) {
        LAUNCH_LDS_T((kg_middle<T, D, MULT_G, NI>), dim3(ma.ntiles + ma.pend.blocks()), op.th_mid, op.lds_mid, op.stream, ma);
        return hipGetLastError();
    }
    if constexpr (sizeof(T) == 8) {
        LAUNCH_LDS_T((kg_middle<T, D, MULT_EM, NI>), dim3(ma.ntiles + ma.pend.blocks()), op.th_mid, op.lds_mid, op.stream, ma);
        return hipGetLastError();
    }
    return hipErrorInvalidValue;
}

template <typename T>
hipError_t gen_middle(const OpPlan& op, const MidArgs<T>& ma, int mult)
{
#define C(N) (op.g.d == 2 ? gen_middle_ni<T, 2, N>(op, ma, mult) : gen_middle_ni<T, 3, N>(op, ma, mult))
    FGH_GEN_NI(op.ni_mid, ma.ax, C);
#undef C
}

#define FGH_GEN_INSTANTIATE(T)                                                             \
    template hipError_t gen_first<T>(const OpPlan&, const FirstArgs<T>&, int, unsigned);   \
    template hipError_t gen_last<T>(const OpPlan&, const LastArgs<T>&, int, unsigned);     \
    template hipError_t gen_lastfirst<T>(const OpPlan&, const LastArgs<T>&, int, unsigned); \
    template hipError_t gen_axis<T>(const OpPlan&, const AxisArgs<T>&, bool, int);         \
    template hipError_t gen_middle<T>(const OpPlan&, const MidArgs<T>&, int);

}  // namespace fgh
