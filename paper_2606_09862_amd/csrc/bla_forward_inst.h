// Launch wrappers of the forward kernels and the list of instantiated shapes.
//
// Shapes: head width D in {32, 64, 128}; padded modes MP in {16, 32, 64, 128};
// padded slots SP in {32, 64, 128, 256} with SP <= max(32, 2 MP).  A shape whose
// LDS tiles exceed the 160 KB of a gfx950 workgroup is reported unsupported.
// Each group of shapes is instantiated in its own translation unit (bla_fwd_*.hip)
// so that the units compile in parallel and can take their own compiler options;
// bla_forward_dispatch.hip selects the instantiation at run time.
#pragma once

#include "bla_forward.h"
#include "bla_forward_pair.h"

#define BLA_FOR_EACH_MS(X, T, D) \
    X(T, D, 16, 32)              \
    X(T, D, 32, 32)              \
    X(T, D, 32, 64)              \
    X(T, D, 64, 32)              \
    X(T, D, 64, 64)              \
    X(T, D, 64, 128)             \
    X(T, D, 128, 32)             \
    X(T, D, 128, 64)             \
    X(T, D, 128, 128)            \
    X(T, D, 128, 256)

#define BLA_FOR_EACH_SHAPE(X, T) \
    BLA_FOR_EACH_MS(X, T, 32)    \
    BLA_FOR_EACH_MS(X, T, 64)    \
    BLA_FOR_EACH_MS(X, T, 128)

namespace bla {

template <typename T, int D, int MP, int SP, int CC = kChunk> constexpr bool fits()
{
    return Fwd<T, D, MP, SP, CC>::LDS_BYTES <= kMaxLds;
}

// Chunk lengths other than the default 64 run on the one-unit kernels and are built for
// M <= 64 (padded modes up to 64), where their tiles and registers fit.
template <int MP, int CC> constexpr bool chunk_built() { return CC == kChunk || MP <= 64; }

// Units per workgroup of the bf16 pair kernel for a shape (0: the shape uses forward_kernel).
template <typename T, int D, int MP, int SP> constexpr int pair_units()
{
    if constexpr (sizeof(T) == 2) {
        return Pair<D, MP, SP>::FITS ? Pair<D, MP, SP>::U : 0;
    } else {
        return 0;
    }
}

// Whether the one-unit forward kernel is built for a shape and chunk length: the pair kernel takes
// every call of 64-token chunks that it exists for.
template <typename T, int D, int MP, int SP, int CC> constexpr bool one_unit_built()
{
    return chunk_built<MP, CC>() && fits<T, D, MP, SP, CC>() && !(CC == kChunk && pair_units<T, D, MP, SP>() > 0);
}

template <typename T, int D, int MP, int SP, int CC>
hipError_t launch_one_unit(const Plan& p, const FwdArgs& a, hipStream_t s)
{
    if constexpr (one_unit_built<T, D, MP, SP, CC>()) {
        const dim3 grid((unsigned)(p.B * p.H * p.nseg));
        if (a.anchor)
            hipLaunchKernelGGL((forward_kernel<T, D, MP, SP, true, CC>), grid, dim3(Geo<T, D, MP, CC>::NTHR), 0, s, a);
        else
            hipLaunchKernelGGL((forward_kernel<T, D, MP, SP, false, CC>), grid, dim3(Geo<T, D, MP, CC>::NTHR), 0, s, a);
        return hipGetLastError();
    } else {
        return hipErrorInvalidValue;
    }
}

template <typename T, int D, int MP, int CC>
hipError_t launch_one_summary(const Plan& p, const FwdArgs& a, hipStream_t s)
{
    // bf16 64-token chunks are summarised by summary_pair_kernel
    if constexpr (chunk_built<MP, CC>() && !(sizeof(T) == 2 && CC == kChunk)) {
        hipLaunchKernelGGL((summary_kernel<T, D, MP, CC>), dim3((unsigned)(p.B * p.H * p.nbs)),
                           dim3(Geo<T, D, MP, CC>::NTHR), 0, s, a);
        return hipGetLastError();
    } else {
        return hipErrorInvalidValue;
    }
}

// Workgroups of the one-unit forward kernel that share a compute unit.
template <typename T, int D, int MP, int SP> int one_unit_wgs(int C)
{
    switch (C) {
    case 16: return Fwd<T, D, MP, SP, 16>::WGS;
    case 32: return Fwd<T, D, MP, SP, 32>::WGS;
    case 64: return Fwd<T, D, MP, SP, 64>::WGS;
    }
    return 1;
}

template <typename T, int D, int MP, int SP> bool one_unit_fits(int C)
{
    switch (C) {
    case 16: return one_unit_built<T, D, MP, SP, 16>();
    case 32: return one_unit_built<T, D, MP, SP, 32>();
    case 64: return one_unit_built<T, D, MP, SP, 64>();
    case 128: return one_unit_built<T, D, MP, SP, 128>();
    }
    return false;
}

template <typename T, int D, int MP, int SP> struct Launch {
    static hipError_t forward(const Plan& p, const FwdArgs& a, hipStream_t s);
    static hipError_t summary(const Plan& p, const FwdArgs& a, hipStream_t s);
};

}  // namespace bla

// Defines the launchers of one shape (used by the bla_fwd_*.hip units).
#define BLA_INSTANTIATE(T, D, MP, SP)                                                                   \
    namespace bla {                                                                                     \
    template <> hipError_t Launch<T, D, MP, SP>::forward(const Plan& p, const FwdArgs& a, hipStream_t s) \
    {                                                                                                   \
        if constexpr (pair_units<T, D, MP, SP>() > 0) {                                                 \
            if (p.pair) {                                                                               \
                constexpr int UU = pair_units<T, D, MP, SP>();                                          \
                dim3 grid((unsigned)((p.B * p.nseg + UU - 1) / UU), (unsigned)p.H);                     \
                if (a.anchor)                                                                           \
                    hipLaunchKernelGGL((forward_pair_kernel<D, MP, SP, true>), grid, dim3(256 * UU), 0, s, a); \
                else                                                                                    \
                    hipLaunchKernelGGL((forward_pair_kernel<D, MP, SP, false>), grid, dim3(256 * UU), 0, s, a); \
                return hipGetLastError();                                                               \
            }                                                                                           \
        }                                                                                               \
        switch (p.C) {                                                                                  \
        case 16: return launch_one_unit<T, D, MP, SP, 16>(p, a, s);                                     \
        case 32: return launch_one_unit<T, D, MP, SP, 32>(p, a, s);                                     \
        case 64: return launch_one_unit<T, D, MP, SP, 64>(p, a, s);                                     \
        case 128: return launch_one_unit<T, D, MP, SP, 128>(p, a, s);                                   \
        }                                                                                               \
        return hipErrorInvalidValue;                                                                    \
    }                                                                                                   \
    template <> hipError_t Launch<T, D, MP, SP>::summary(const Plan& p, const FwdArgs& a, hipStream_t s) \
    {                                                                                                   \
        if constexpr (pair_units<T, D, MP, SP>() > 0) {                                                 \
            if (p.pair && p.enter == kEnterPass) {                                                      \
                const dim3 sgrid((unsigned)state_pass_grid<D, MP>((long long)p.B * p.H));               \
                if (p.cps == 1)                                                                         \
                    hipLaunchKernelGGL((state_pair_kernel<D, MP, true>), sgrid, dim3(StatePass<D, MP>::NTHR), 0, s, a);  \
                else                                                                                    \
                    hipLaunchKernelGGL((state_pair_kernel<D, MP, false>), sgrid, dim3(StatePass<D, MP>::NTHR), 0, s, a); \
                return hipGetLastError();                                                               \
            }                                                                                           \
            if (p.pair) {                                                                               \
                hipLaunchKernelGGL((summary_pair_kernel<D, MP>),                                        \
                                   dim3((unsigned)summary_grid_x<D, MP>((long long)p.B * p.nbs), (unsigned)p.H),  \
                                   dim3(summary_threads<D, MP>()), 0, s, a);                            \
                return hipGetLastError();                                                               \
            }                                                                                           \
        }                                                                                               \
        if constexpr (sizeof(T) == 2 && pair_units<T, D, MP, SP>() == 0) {                              \
            if (p.C == kChunk) { /* bf16, 64-token chunks: the sliced summary kernel */                 \
                hipLaunchKernelGGL((summary_pair_kernel<D, MP, true>),                                  \
                                   dim3((unsigned)summary_grid_x<D, MP>((long long)p.B * p.nbs), (unsigned)p.H),  \
                                   dim3(summary_threads<D, MP>()), 0, s, a);                            \
                return hipGetLastError();                                                               \
            }                                                                                           \
        }                                                                                               \
        switch (p.C) {                                                                                  \
        case 16: return launch_one_summary<T, D, MP, 16>(p, a, s);                                      \
        case 32: return launch_one_summary<T, D, MP, 32>(p, a, s);                                      \
        case 64: return launch_one_summary<T, D, MP, 64>(p, a, s);                                      \
        case 128: return launch_one_summary<T, D, MP, 128>(p, a, s);                                    \
        }                                                                                               \
        return hipErrorInvalidValue;                                                                    \
    }                                                                                                   \
    }
