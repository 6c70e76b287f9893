// Whole Lanczos runs of a few columns inside one workgroup, for matrices
// whose v_j column fits in LDS (up to about 39 000 rows in FP32, 19 000 in
// FP64).  Columns never meet in the recurrence, so a workgroup needs nothing
// from another one: it makes its probe columns, runs every step and leaves
// the coefficients, with no pass over memory for the vectors and no launch
// or grid-wide wait between steps.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <type_traits>

#include "lanczos_device.h"
#include "resident.h"
#include "wave_device.h"

namespace vne {

namespace {

// The lane's rows' entries of v_{j-1} (then of w), in registers: vectors with
// a wave-uniform index (the register file is indexed directly).  An index
// past its vector would reach other registers, so the rounds of the two
// vectors are loops of their own (for_rounds), never a choice by index.
// BIG: as many as a layout may have; otherwise the few of a small matrix,
// which leaves the registers to the serial part of a step (measured: with the
// big vectors there, spills cost 2 us a step at n = 2000).
template <typename T, bool BIG> struct Slots;
template <> struct Slots<float, true> {
    typedef float A __attribute__((ext_vector_type(32)));
    typedef float B __attribute__((ext_vector_type(8)));
    static constexpr int NA = 32, NB = 8;
};
template <> struct Slots<double, true> {
    typedef double A __attribute__((ext_vector_type(16)));
    typedef double B __attribute__((ext_vector_type(4)));
    static constexpr int NA = 16, NB = 4;
};
template <> struct Slots<float, false> {
    typedef float A __attribute__((ext_vector_type(8)));
    typedef float B __attribute__((ext_vector_type(2)));
    static constexpr int NA = 8, NB = 0;
};
template <> struct Slots<double, false> {
    typedef double A __attribute__((ext_vector_type(4)));
    typedef double B __attribute__((ext_vector_type(2)));
    static constexpr int NA = 4, NB = 0;
};
static_assert(kResidentSlots32 <= Slots<float, true>::NA + Slots<float, true>::NB, "slots of an FP32 lane");
static_assert(kResidentSlots64 <= Slots<double, true>::NA + Slots<double, true>::NB, "slots of an FP64 lane");

template <typename T, int C> struct Cols {
    typedef T type __attribute__((ext_vector_type(C)));
};
template <typename T> struct Pair;
template <> struct Pair<float> { using type = float2; };
template <> struct Pair<double> { using type = double2; };

// Sums of N values per thread over the workgroup, returned in every lane of
// wave 0 (fixed order: lanes, then waves).  Every wave has passed a barrier.
// red: [N][16].
template <int N>
__device__ __forceinline__ void group_totals(const double (&v)[N], double (&out)[N], double *red, int wave, int lane,
                                             int waves) {
#pragma unroll
    for (int q = 0; q < N; ++q) {
        const double t = wave_total(v[q]);
        if (lane == 63) red[q * 16 + wave] = t;
    }
    lds_barrier();
    if (wave != 0) return;
    // lane 16 i + w holds wave w's share of value q + i: rows of 16 lanes
    double t[(N + 3) / 4];
#pragma unroll
    for (int q = 0; q < N; q += 4) {
        const int mine = q + (lane >> 4);
        t[q / 4] = mine < N && (lane & 15) < waves ? red[mine * 16 + (lane & 15)] : 0.0;
    }
#pragma unroll
    for (int q = 0; q < N; q += 4) {
        double &x = t[q / 4];
        x = dpp_add<0x111, 0xf>(x);
        x = dpp_add<0x112, 0xf>(x);
        x = dpp_add<0x114, 0xf>(x);
        x = dpp_add<0x118, 0xf>(x);
    }
#pragma unroll
    for (int q = 0; q < N; ++q) out[q] = from_lane(t[q / 4], (q & 3) * 16 + 15);
}

// v[c] for lane c
template <int C>
__device__ __forceinline__ double by_lane(const double (&v)[C], int lane) {
    double x = v[0];
#pragma unroll
    for (int c = 1; c < C; ++c) x = lane == c ? v[c] : x;
    return x;
}

// What bounds it: the LDS gathers (one 64-lane read of v_j per 64 stored
// entries and group of C columns) and the FP64 additions behind them; the
// matrix is read from L2 once per step and group (2 bytes an entry when the
// off-diagonal values are all equal, as in a Laplacian).
template <typename T, int C, bool UNIT, bool BIG>
__device__ __forceinline__ void run_columns(const ResidentJob J, int col0) {
    using Vec = typename Cols<T, C>::type;
    using VPair = typename Pair<T>::type;
    extern __shared__ char lds[];
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int waves = blockDim.x >> 6;
    const int R = J.rounds, P = J.positions;
    Vec *V = reinterpret_cast<Vec *>(lds);
    double *red = reinterpret_cast<double *>(lds + ((((size_t)P + 1) * sizeof(Vec) + 15) & ~(size_t)15));
    double *bc = red + (size_t)16 * 3 * C;      // alpha, 1 / beta and beta of the step, per column
    const uint32_t lds0 = (uint32_t)(uintptr_t)(VNE_LDS char *)lds;
    const VNE_GLOBAL uint32_t *words = global<uint32_t>(J.words);
    const VNE_GLOBAL VPair *vals = global<VPair>(J.vals);
    const VNE_GLOBAL int32_t *row_of = global<int32_t>(J.row_of);
    const VNE_GLOBAL double *diag = global<double>(J.diag);
    const VNE_GLOBAL int2 *spans = global<int2>(J.spans);
    const int base = wave * R * 64 + lane;
    using S = Slots<T, BIG>;
    typename S::A slot_a = (T)0;
    typename S::B slot_b = (T)0;
    // body(round, slots, index of the round's first slot) for every round
    // (R * C <= NA + NB: the host's limit)
    // (unrolled no further than this: wider, the slots spill)
    auto for_rounds = [&](auto body) {
        constexpr int RA = S::NA / C;
#pragma unroll 1
        for (int r = 0; r < (S::NB > 0 ? min(R, RA) : R); ++r) body(r, slot_a, r * C);
        if constexpr (S::NB > 0)
#pragma unroll 1
            for (int r = RA; r < R; ++r) body(r, slot_b, (r - RA) * C);
    };

    if (threadIdx.x == 0) V[P] = (Vec)(T)0;
    // probe columns: raw values, then centred (Remark 4.6), ||c||^2 of the
    // stored values, v_1 = c / ||c||
    {
        double s[C];
#pragma unroll
        for (int c = 0; c < C; ++c) s[c] = 0.0;
        for_rounds([&](int r, auto &slot, int i0) {
            const int row = row_of[base + r * 64];
#pragma unroll
            for (int c = 0; c < C; ++c) {
                double b = 0.0;
                if (row >= 0 && col0 + c < J.m) {
                    if (J.gen == GEN_RADEMACHER)
                        b = rademacher(J.seed, global<int64_t>(J.keys)[row], (int64_t)J.col_offset + col0 + c);
                    else if (J.gen == GEN_COLORING)
                        b = global<int32_t>(J.colors)[row] == col0 + c ? 1.0 : 0.0;
                    else
                        b = (double)global<T>(J.dense)[(int64_t)row * J.ld_dense + col0 + c];
                }
                slot[i0 + c] = (T)b;
                s[c] += b;
            }
        });
        double t[C];
        group_totals<C>(s, t, red, wave, lane, waves);
        if (wave == 0 && lane < C) bc[lane] = J.desing ? by_lane<C>(t, lane) / (double)J.n : 0.0;
        lds_barrier();
        double mu[C];
#pragma unroll
        for (int c = 0; c < C; ++c) {
            mu[c] = bc[c];
            s[c] = 0.0;
        }
        for_rounds([&](int r, auto &slot, int i0) {
            const int row = row_of[base + r * 64];
#pragma unroll
            for (int c = 0; c < C; ++c) {
                const T x = row >= 0 && col0 + c < J.m ? (T)((double)slot[i0 + c] - mu[c]) : (T)0;
                slot[i0 + c] = x;
                s[c] += (double)x * (double)x;
            }
        });
        group_totals<C>(s, t, red, wave, lane, waves);
        if (wave == 0 && lane < C) {
            const int col = col0 + lane;
            const double tc = by_lane<C>(t, lane);
            double inv = 0.0;
            if (!isfinite(tc) && col < J.m) atomicOr(J.flags, 1);
            if (tc > 0.0 && isfinite(tc) && col < J.m) inv = 1.0 / sqrt(tc);
            J.norm2[col] = tc;
            J.k_eff[col] = inv != 0.0 ? J.k : 0;
            bc[lane] = 0.0;
            bc[C + lane] = inv;
            bc[2 * C + lane] = 0.0;
        }
        lds_barrier();
    }
    {
        T inv[C];
#pragma unroll
        for (int c = 0; c < C; ++c) inv[c] = (T)bc[C + c];
        for_rounds([&](int r, auto &slot, int i0) {
            Vec v;
#pragma unroll
            for (int c = 0; c < C; ++c) {
                v[c] = materialize((T)slot[i0 + c], (T)0, (T)0, inv[c]);
                slot[i0 + c] = (T)0;
            }
            V[base + r * 64] = v;
        });
    }
    lds_barrier();

    // Gathers of a slice run GW words (2 GW reads of v_j a lane) at a time,
    // PF words of the next slice are loaded while this one runs.
    constexpr int GW = C == 4 ? 2 : 4, PF = UNIT && sizeof(Vec) <= 8 && (!BIG || sizeof(T) == 4) ? 8 : 4;
    uint32_t nw[PF];
    VPair nx[PF];
#pragma unroll
    for (int i = 0; i < PF; ++i) {
        nw[i] = 0;
        nx[i] = VPair{(T)0, (T)0};
    }
    // the wave's slices, one a lane (R <= 64), read back by round
    int4 mine = make_int4(0, 0, 0, 0);
    if (lane < R) {
        const VNE_GLOBAL int32_t *sl = global<int32_t>(J.slices) + ((size_t)wave * R + lane) * 4;
        mine = make_int4(sl[0], sl[1], sl[2], sl[3]);
    }
    // word rows row64 + i: one 32-bit offset from a scalar base, the rows by
    // the instruction's own offset (the arrays end in spare rows, so that a
    // slice's last group may read past it)
    const unsigned at = (unsigned)lane;
    auto load = [&](uint32_t *w, VPair *x, int row64, auto count) {
        constexpr int N = decltype(count)::value;
        const VNE_GLOBAL char *wp = (const VNE_GLOBAL char *)words + ((unsigned)row64 * 256u + at * 4u);
#pragma unroll
        for (int i = 0; i < N; ++i) w[i] = *(const VNE_GLOBAL uint32_t *)(wp + 256 * i);
        if (!UNIT) {
            constexpr unsigned es = sizeof(VPair);
            const VNE_GLOBAL char *xp = (const VNE_GLOBAL char *)vals + ((unsigned)row64 * (64u * es) + at * es);
#pragma unroll
            for (int i = 0; i < N; ++i) {
                const VNE_GLOBAL T *p = (const VNE_GLOBAL T *)(xp + 64 * es * i);
                x[i] = VPair{p[0], p[1]};
            }
        }
    };
    using One = std::integral_constant<int, 1>;
    using Two = std::integral_constant<int, 2>;
    using Four = std::integral_constant<int, 4>;
    using Group = std::integral_constant<int, GW>;
    // the first words of round r's slice (a short one)
    double next_diag = 0.0;
    auto fetch = [&](int r) {
        if (UNIT) next_diag = (diag + (size_t)(unsigned)((wave * R + r) * 64))[at];
        if (__builtin_amdgcn_readlane(mine.x, r) != 1) return;
        const int first = __builtin_amdgcn_readlane(mine.y, r), len = __builtin_amdgcn_readlane(mine.z, r);
#pragma unroll
        for (int g = 0; g < PF; g += 4)
            if (g < len) load(nw + g, nx + g, first + g, Four{});
    };
    // the entries of N words: 2 N gathers in flight, `between` while they
    // are, then their sums
    auto add = [&](auto n_words, const uint32_t *w, const VPair *x, double (&acc)[C], auto between) {
        constexpr int N = decltype(n_words)::value;
        Vec a[N], b[N];
        VPair y[N];
#pragma unroll
        for (int i = 0; i < N; ++i) {
            a[i] = *(const VNE_LDS Vec *)(uintptr_t)half_times<0, (int)sizeof(Vec)>(w[i], lds0);
            b[i] = *(const VNE_LDS Vec *)(uintptr_t)half_times<1, (int)sizeof(Vec)>(w[i], lds0);
            y[i] = x[i];
        }
        between();
#pragma unroll
        for (int i = 0; i < N; ++i)
#pragma unroll
            for (int c = 0; c < C; ++c) {
                if (UNIT) {
                    acc[c] += (double)a[i][c];
                    acc[c] += (double)b[i][c];
                } else {
                    acc[c] = fma((double)y[i].x, (double)a[i][c], acc[c]);
                    acc[c] = fma((double)y[i].y, (double)b[i][c], acc[c]);
                }
            }
    };
    auto nothing = [] {};
    const double scaled_off = J.scale * J.off_value;
    fetch(0);
    for (int j = 1; j <= J.k; ++j) {
        double coup[C], s[3 * C];
#pragma unroll
        for (int c = 0; c < C; ++c) coup[c] = bc[2 * C + c];
#pragma unroll
        for (int q = 0; q < 3 * C; ++q) s[q] = 0.0;
        for_rounds([&](int r, auto &slot, int i0) {
            double acc[C];
#pragma unroll
            for (int c = 0; c < C; ++c) acc[c] = 0.0;
            double dg = 0.0;
            if (UNIT) dg = next_diag;
            const int kind = __builtin_amdgcn_readlane(mine.x, r), first = __builtin_amdgcn_readlane(mine.y, r);
            const int len = __builtin_amdgcn_readlane(mine.z, r);
            const int next = r + 1 < R ? r + 1 : 0;        // round 0 again: the next step's
            if (kind == 1) {
                // the next slice's words replace this one's as soon as their
                // last gathers are issued
                auto ahead = [&] { fetch(next); };
#pragma unroll
                for (int g = 0; g < PF; g += GW) {
                    const bool last = g + GW >= len && len <= PF;
                    if (g + GW < len || (g + GW == len && !last)) add(Group{}, nw + g, nx + g, acc, nothing);
                    else if (g + GW == len) add(Group{}, nw + g, nx + g, acc, ahead);
                    else if (GW == 4 && g + 2 == len) add(Two{}, nw + g, nx + g, acc, ahead);
                }
                if (len > PF) {
                    // the rest of a longer slice, the next group in flight
                    uint32_t cw[GW];
                    VPair cx[GW];
                    load(cw, cx, first + PF, Group{});
                    for (int t = PF; t < len; t += GW) {
                        uint32_t w[GW];
                        VPair x[GW];
#pragma unroll
                        for (int i = 0; i < GW; ++i) {
                            w[i] = cw[i];
                            x[i] = cx[i];
                        }
                        if (t + GW < len) load(cw, cx, first + t + GW, Group{});
                        if (t + GW <= len) add(Group{}, w, x, acc, nothing);
                        else add(Two{}, w, x, acc, nothing);
                    }
                    fetch(next);
                } else if (len == 0) {
                    fetch(next);
                }
            } else if (kind == 2) {
                // long rows, entries over the lanes, LB rows at a time
                constexpr int LB = sizeof(Vec) <= 8 ? 4 : 2;
                const int rows = __builtin_amdgcn_readlane(mine.w, r);
                const VNE_GLOBAL int32_t *sp = (const VNE_GLOBAL int32_t *)(spans + first + min(lane, rows - 1));
                const int2 span = make_int2(sp[0], sp[1]);
                for (int q0 = 0; q0 < rows; q0 += LB) {
                    uint32_t w[LB];
                    VPair x[LB];
                    double part[LB][C];
#pragma unroll
                    for (int i = 0; i < LB; ++i)
                        load(w + i, x + i, __builtin_amdgcn_readlane(span.x, min(q0 + i, rows - 1)), One{});
#pragma unroll
                    for (int i = 0; i < LB; ++i) {
#pragma unroll
                        for (int c = 0; c < C; ++c) part[i][c] = 0.0;
                        add(One{}, w + i, x + i, part[i], nothing);
                    }
#pragma unroll
                    for (int i = 0; i < LB; ++i) {
                        const int q = min(q0 + i, rows - 1);
                        const int a0 = __builtin_amdgcn_readlane(span.x, q);
                        const int cnt = __builtin_amdgcn_readlane(span.y, q);
                        for (int t = 1; t < cnt; ++t) {
                            load(w + i, x + i, a0 + t, One{});
                            add(One{}, w + i, x + i, part[i], nothing);
                        }
                    }
#pragma unroll
                    for (int i = 0; i < LB; ++i)
#pragma unroll
                        for (int c = 0; c < C; ++c) {
                            const double tot = from_lane(wave_total(part[i][c]), 63);
                            acc[c] = lane == q0 + i && q0 + i < rows ? tot : acc[c];
                        }
                }
                fetch(next);
            } else {
                fetch(next);
            }
            // w = scale (A v_j) - beta_{j-1} v_{j-1}
            const Vec v = V[base + r * 64];
            const double sd = J.scale * dg;
#pragma unroll
            for (int c = 0; c < C; ++c) {
                const double vd = (double)v[c];
                const double u = UNIT ? fma(sd, vd, scaled_off * acc[c]) : J.scale * acc[c];
                const T w = (T)fma(-coup[c], (double)slot[i0 + c], u);
                slot[i0 + c] = w;
                const double wd = (double)w;
                s[c] = fma(vd, wd, s[c]);
                s[C + c] = fma(wd, wd, s[C + c]);
                s[2 * C + c] = fma(vd, vd, s[2 * C + c]);
            }
        });
        double tot[3 * C];
        group_totals<3 * C>(s, tot, red, wave, lane, waves);
        if (wave == 0) {
            // alpha, beta, breakdown and the scalars of v_{j+1} (as
            // update_coefficients does for the launched steps)
            const int c = lane, col = col0 + lane;
            double a3[3][C];
#pragma unroll
            for (int i = 0; i < C; ++i) {
                a3[0][i] = tot[i];
                a3[1][i] = tot[C + i];
                a3[2][i] = tot[2 * C + i];
            }
            const double svw = by_lane<C>(a3[0], lane), sww = by_lane<C>(a3[1], lane), svv = by_lane<C>(a3[2], lane);
            if (lane < C) {
                const double inv_prev = bc[C + c], coup_prev = bc[2 * C + c];
                double alpha = 0.0, beta = 0.0, al = 0.0, inv = 0.0, cp = 0.0;
                if (inv_prev != 0.0) {
                    alpha = svw / svv;
                    double b2 = sww - alpha * svw;
                    b2 = b2 > 0.0 ? b2 : 0.0;
                    const double b = sqrt(b2);
                    const bool finite = isfinite(alpha) && isfinite(b);
                    if (!finite) atomicOr(J.flags, 1);
                    if (!finite || b <= J.tau * (fabs(alpha) + coup_prev)) {
                        J.k_eff[col] = j;
                    } else {
                        beta = b;
                        if (j < J.k) {
                            al = alpha;
                            inv = 1.0 / b;
                            cp = b;
                        }
                    }
                }
                J.alpha[(int64_t)col * J.ld_k + j - 1] = alpha;
                J.beta[(int64_t)col * J.ld_k + j - 1] = beta;
                bc[c] = al;
                bc[C + c] = inv;
                bc[2 * C + c] = cp;
            }
        }
        lds_barrier();
        T al[C], inv[C];
        bool live = false;
#pragma unroll
        for (int c = 0; c < C; ++c) {
            al[c] = (T)bc[c];
            inv[c] = (T)bc[C + c];
            live = live || bc[C + c] != 0.0;
        }
        if (!live) {                               // broken down (or done): the rest is zero
            if (wave == 0 && lane < C)
                for (int jj = j; jj < J.k; ++jj) {
                    J.alpha[(int64_t)(col0 + lane) * J.ld_k + jj] = 0.0;
                    J.beta[(int64_t)(col0 + lane) * J.ld_k + jj] = 0.0;
                }
            break;
        }
        for_rounds([&](int r, auto &slot, int i0) {
            const Vec v = V[base + r * 64];
            Vec nv;
#pragma unroll
            for (int c = 0; c < C; ++c) {
                nv[c] = materialize((T)slot[i0 + c], v[c], al[c], inv[c]);
                slot[i0 + c] = v[c];
            }
            V[base + r * 64] = nv;
        });
        lds_barrier();
    }
}

template <typename T, int C, bool UNIT, bool BIG>
__global__ void __launch_bounds__(1024) k_resident_one(ResidentJob job) {
    run_columns<T, C, UNIT, BIG>(job, blockIdx.x * C);
}

template <typename T, int C, bool UNIT, bool BIG>
__global__ void __launch_bounds__(1024) k_resident_many(const ResidentJob *jobs, const int2 *map) {
    const int2 e = map[blockIdx.x];
    const int job = __builtin_amdgcn_readfirstlane(e.x);
    if (job < 0) return;
    const ResidentJob j = jobs[job];
    run_columns<T, C, UNIT, BIG>(j, __builtin_amdgcn_readfirstlane(e.y));
}

struct Launch {
    const ResidentJob *one, *jobs;
    const int2 *map;
    unsigned grid;
    int waves;
    size_t lds;
    hipStream_t s;
    ResidentKind kind;
};

template <typename T, int C, bool UNIT, bool BIG>
hipError_t launch(const Launch &l) {
    const void *f = l.one ? (const void *)k_resident_one<T, C, UNIT, BIG> : (const void *)k_resident_many<T, C, UNIT, BIG>;
    const hipError_t e = hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, (int)kResidentLds);
    if (e != hipSuccess) return e;
    if (l.one)
        hipLaunchKernelGGL((k_resident_one<T, C, UNIT, BIG>), dim3(l.grid), dim3(64 * l.waves), l.lds, l.s, *l.one);
    else
        hipLaunchKernelGGL((k_resident_many<T, C, UNIT, BIG>), dim3(l.grid), dim3(64 * l.waves), l.lds, l.s, l.jobs,
                           l.map);
    return hipGetLastError();
}

// (two FP64 columns take equal off-diagonal values only)
template <typename T, int C>
hipError_t launch_cols(const Launch &l) {
    if (l.kind.unit) return l.kind.big ? launch<T, C, true, true>(l) : launch<T, C, true, false>(l);
    if constexpr (sizeof(T) == 4 || C == 1)
        return l.kind.big ? launch<T, C, false, true>(l) : launch<T, C, false, false>(l);
    return hipErrorInvalidValue;
}

hipError_t launch_kind(const Launch &l) {
    if (l.lds > kResidentLds || l.waves < 1 || l.waves > 16) return hipErrorInvalidValue;
    if (l.kind.fp64) {
        if (l.kind.cols == 1) return launch_cols<double, 1>(l);
        if (l.kind.cols == 2) return launch_cols<double, 2>(l);
    } else {
        if (l.kind.cols == 1) return launch_cols<float, 1>(l);
        if (l.kind.cols == 2) return launch_cols<float, 2>(l);
        if (l.kind.cols == 4) return launch_cols<float, 4>(l);
    }
    return hipErrorInvalidValue;
}

}  // namespace

size_t resident_lds(int positions, int cols, bool fp64) {
    const size_t v = ((size_t)positions + 1) * cols * (fp64 ? 8 : 4);
    return ((v + 15) & ~(size_t)15) + ((size_t)16 * 3 * cols + 3 * cols) * 8;
}

ResidentKind resident_kind(int rounds, int cols, bool unit, bool fp64) {
    const int few = fp64 ? Slots<double, false>::NA : Slots<float, false>::NA;
    return ResidentKind{cols, unit, fp64, rounds * cols > few};
}

hipError_t launch_resident_one(const ResidentJob &job, int waves, const ResidentKind &kind, hipStream_t s) {
    return launch_kind(Launch{&job, nullptr, nullptr, (unsigned)((job.m + kind.cols - 1) / kind.cols), waves,
                              resident_lds(job.positions, kind.cols, kind.fp64), s, kind});
}

hipError_t launch_resident_many(const ResidentJob *jobs, const int2 *map, int32_t entries, int waves,
                                const ResidentKind &kind, size_t lds, hipStream_t s) {
    if (entries <= 0) return hipSuccess;
    return launch_kind(Launch{nullptr, jobs, map, (unsigned)entries, waves, lds, s, kind});
}

}  // namespace vne
