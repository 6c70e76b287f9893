// Rational Arnoldi steps of small matrices, one workgroup per column: the
// product, the projection, the conjugate-gradient solve and the
// orthogonalization each run from LDS and registers in one launch.  Launched
// over the whole block they were six kernels and two reductions of 512 partials
// an iteration of conjugate gradients (128 us on a 40 x 40 grid); here an
// iteration is one pass over the column's rows and two sums over the
// workgroup (about 3 us there, bound by the chain gathers - sum - barrier -
// sum - barrier of one column).  40 x 40 grid, 4 columns, 7 steps: 35.5 ms
// before, 0.91 ms now.
//
// Taken wherever the layout fits in kRChipRounds rounds of registers: slower
// at no size or density measured (times of 12 steps launched with the parallel
// reduction and here: 100 rows of 4 entries, 1 column 11.7 and 1.0 ms; 5000
// rows, 64 columns 21.9 and 2.9; 5000 rows of 500, 1 column 61.8 and 14.5, 64
// columns 51.3 and 15.2; 2000 rows of 1000, 8 columns 43.1 and 15.8).
#include <hip/hip_runtime.h>

#include <cmath>

#include "rational_chip.h"
#include "resident.h"
#include "wave_device.h"

namespace vne {

namespace {

constexpr int RM = kRChipRounds;

struct Lanes {
    int lane, wave, waves;
    __device__ __forceinline__ Lanes()
        : lane(threadIdx.x & 63), wave(__builtin_amdgcn_readfirstlane(threadIdx.x >> 6)), waves(blockDim.x >> 6) {}
};

// sum over the workgroup in every thread (fixed order).  red: 16 doubles that
// the call before last may still have been read from.
__device__ __forceinline__ double block_sum(double v, double *red, const Lanes &l) {
    const double t = wave_total(v);
    if (l.lane == 63) red[l.wave] = t;
    lds_barrier();
    double s = (l.lane & 15) < l.waves ? red[l.lane & 15] : 0.0;
    s = dpp_add<0x111, 0xf>(s);
    s = dpp_add<0x112, 0xf>(s);
    s = dpp_add<0x114, 0xf>(s);
    s = dpp_add<0x118, 0xf>(s);
    return from_lane(s, 15);
}

// N sums at once; out[q] (LDS, N doubles) is ready after the caller's next
// barrier.  red: [N][16].
template <int N>
__device__ __forceinline__ void block_sums(const double (&v)[N], int count, double *red, double *out, const Lanes &l) {
#pragma unroll
    for (int q = 0; q < N; ++q) {
        const double t = wave_total(v[q]);
        if (l.lane == 63) red[q * 16 + l.wave] = t;
    }
    lds_barrier();
    for (int q = l.wave; q < count; q += l.waves) {
        double s = (l.lane & 15) < l.waves ? red[q * 16 + (l.lane & 15)] : 0.0;
        s = dpp_add<0x111, 0xf>(s);
        s = dpp_add<0x112, 0xf>(s);
        s = dpp_add<0x114, 0xf>(s);
        s = dpp_add<0x118, 0xf>(s);
        if (l.lane == 15) out[q] = s;
    }
}

// (scale A x) at the thread's row of round r; x: LDS, positions() + 1 entries
// with a zero behind the last; words from LDS (IN_LDS) or device memory.
template <bool UNIT, bool IN_LDS>
__device__ __forceinline__ double product(const RChip &a, int r, const double *x, const uint32_t *lds_words,
                                          const Lanes &l) {
    const int32_t *sl = a.slices + 4 * (l.wave * a.rounds + r);
    const int kind = sl[0], first = sl[1], len = sl[2], rows = sl[3];
    const uint32_t *words = IN_LDS ? lds_words : a.words;
    auto one = [&](int64_t o, double &acc) {
        const uint32_t w = words[o];
        const double u = x[w & 0xffffu], v = x[w >> 16];
        if (UNIT) {
            acc += u;
            acc += v;
        } else {
            acc = fma(a.vals[2 * o], u, acc);
            acc = fma(a.vals[2 * o + 1], v, acc);
        }
    };
    double acc = 0.0;
    if (kind == 1) {
        for (int t = 0; t < len; t += 2) {       // an even number of words
            one((int64_t)(first + t) * 64 + l.lane, acc);
            one((int64_t)(first + t + 1) * 64 + l.lane, acc);
        }
    } else if (kind == 2) {
        for (int q = 0; q < rows; ++q) {
            const int a0 = a.spans[2 * (first + q)], cnt = a.spans[2 * (first + q) + 1];
            double part = 0.0;
            for (int t = 0; t < cnt; ++t) one((int64_t)(a0 + t) * 64 + l.lane, part);
            const double tot = from_lane(wave_total(part), 63);
            acc = l.lane == q ? tot : acc;
        }
    }
    if (!UNIT) return a.scale * acc;
    const int p = (l.wave * a.rounds + r) * 64 + l.lane;
    return a.scale * fma(a.diag[p], x[p], a.off_value * acc);
}

// v_{j+1} = w / ||w||, or 0 where w lost all but 1e-12 of its norm (an
// invariant subspace: the basis stops growing)
__device__ __forceinline__ bool grows(double ww, double ww0) { return ww > 1e-24 * ww0 && ww > 0.0; }

__global__ void __launch_bounds__(1024) k_rchip_start(RChip a, const double *W0, int32_t mp, const double *norm2) {
    const int c = blockIdx.x;
    const double s = norm2[c];
    for (int p = threadIdx.x; p < a.positions; p += blockDim.x) {
        const int row = a.row_of[p];
        a.V[(int64_t)c * a.kb * a.positions + p] = row >= 0 && grows(s, s) ? W0[(int64_t)row * mp + c] / sqrt(s) : 0.0;
    }
}

template <bool UNIT>
__global__ void __launch_bounds__(1024) k_rchip_project(RChip a, int32_t j, double *H) {
    extern __shared__ double lds[];
    const Lanes l;
    const int c = blockIdx.x, P = a.positions;
    double *x = lds, *red = lds + P + 1, *out = red + 2 * 8 * 16;
    const double *V = a.V + (int64_t)c * a.kb * P;
    const int base = l.wave * a.rounds * 64 + l.lane;
    for (int r = 0; r < a.rounds; ++r) x[base + r * 64] = V[(int64_t)(j - 1) * P + base + r * 64];
    if (threadIdx.x == 0) x[P] = 0.0;
    lds_barrier();
    double u[RM];
#pragma unroll
    for (int r = 0; r < RM; ++r) {
        u[r] = 0.0;
        if (r < a.rounds) {
            u[r] = product<UNIT, false>(a, r, x, nullptr, l);
            a.U[(int64_t)c * P + base + r * 64] = u[r];
        }
    }
    for (int b0 = 0, turn = 0; b0 < j; b0 += 8, turn ^= 1) {
        double d[8];
#pragma unroll
        for (int q = 0; q < 8; ++q) {
            d[q] = 0.0;
            if (b0 + q < j)
#pragma unroll
                for (int r = 0; r < RM; ++r)
                    if (r < a.rounds) d[q] = fma(V[(int64_t)(b0 + q) * P + base + r * 64], u[r], d[q]);
        }
        block_sums<8>(d, min(8, j - b0), red + turn * 8 * 16, out + b0, l);
    }
    lds_barrier();
    for (int i = threadIdx.x; i < j; i += blockDim.x) {
        H[((int64_t)c * a.kb + i) * a.kb + (j - 1)] = out[i];
        H[((int64_t)c * a.kb + (j - 1)) * a.kb + i] = out[i];
    }
}

template <bool UNIT, bool IN_LDS>
__global__ void __launch_bounds__(1024) k_rchip_solve(RChip a, const double *xi, double tol2, int32_t cg_max,
                                                      int32_t *iters, int64_t *apps) {
    extern __shared__ double lds[];
    const Lanes l;
    const int c = blockIdx.x, P = a.positions;
    const int base = l.wave * a.rounds * 64 + l.lane;
    double *x = lds, *red = lds + P + 1;                  // x: the direction p
    uint32_t *words = (uint32_t *)(red + 32);
    const double *U = a.U + (int64_t)c * P;
    double *W = a.W + (int64_t)c * P;
    const double xc = xi[c];
    if (xc == 0.0) {
        for (int r = 0; r < a.rounds; ++r) W[base + r * 64] = U[base + r * 64];
        return;
    }
    const double inv = 1.0 / xc;
    if (IN_LDS)
        for (int t = threadIdx.x; t < a.word_rows * 64; t += blockDim.x) words[t] = a.words[t];
    double sol[RM], res[RM], dir[RM], q[RM];
    double part = 0.0;
#pragma unroll
    for (int r = 0; r < RM; ++r) {
        sol[r] = q[r] = 0.0;
        res[r] = r < a.rounds ? U[base + r * 64] : 0.0;
        dir[r] = res[r];
        if (r < a.rounds) x[base + r * 64] = dir[r];
        part = fma(res[r], res[r], part);
    }
    if (threadIdx.x == 0) x[P] = 0.0;
    double rr = block_sum(part, red, l);
    const double rr0 = rr;
    int it = 0;
    // a zero right-hand side is solved by 0 and counts no iteration
    while (rr0 != 0.0) {
        part = 0.0;
#pragma unroll
        for (int r = 0; r < RM; ++r)
            if (r < a.rounds) {
                q[r] = fma(-product<UNIT, IN_LDS>(a, r, x, words, l), inv, dir[r]);
                part = fma(dir[r], q[r], part);
            }
        const double pq = block_sum(part, red + 16, l);
        const double alpha = pq != 0.0 ? rr / pq : 0.0;
        part = 0.0;
#pragma unroll
        for (int r = 0; r < RM; ++r) {
            sol[r] = fma(alpha, dir[r], sol[r]);
            res[r] = fma(-alpha, q[r], res[r]);
            part = fma(res[r], res[r], part);
        }
        const double rn = block_sum(part, red, l);
        ++it;
        const double beta = rr > 0.0 ? rn / rr : 0.0;
        rr = rn;
        if (!(rn > tol2 * rr0) || it >= cg_max) break;
#pragma unroll
        for (int r = 0; r < RM; ++r) {
            dir[r] = fma(beta, dir[r], res[r]);
            if (r < a.rounds) x[base + r * 64] = dir[r];
        }
        lds_barrier();
    }
#pragma unroll
    for (int r = 0; r < RM; ++r)
        if (r < a.rounds) W[base + r * 64] = sol[r];
    if (threadIdx.x == 0) {
        iters[c] += it;
        apps[c] += it;
    }
}

__global__ void __launch_bounds__(1024) k_rchip_orthogonalize(RChip a, int32_t j, int32_t from_u, int32_t commit,
                                                              double *ww, double *ww0, int32_t *ke) {
    extern __shared__ double lds[];
    const Lanes l;
    const int c = blockIdx.x, P = a.positions;
    const int base = l.wave * a.rounds * 64 + l.lane;
    double *red = lds, *h = red + 2 * 8 * 16, *red1 = h + 64;
    const double *V = a.V + (int64_t)c * a.kb * P;
    const double *src = (from_u ? a.U : a.W) + (int64_t)c * P;
    double w[RM], part = 0.0;
#pragma unroll
    for (int r = 0; r < RM; ++r) {
        w[r] = r < a.rounds ? src[base + r * 64] : 0.0;
        part = fma(w[r], w[r], part);
    }
    const double before = block_sum(part, red1, l);
    for (int pass = 0; pass < 2; ++pass) {
        for (int b0 = 0, turn = 0; b0 < j; b0 += 8, turn ^= 1) {
            double d[8];
#pragma unroll
            for (int q = 0; q < 8; ++q) {
                d[q] = 0.0;
                if (b0 + q < j)
#pragma unroll
                    for (int r = 0; r < RM; ++r)
                        if (r < a.rounds) d[q] = fma(V[(int64_t)(b0 + q) * P + base + r * 64], w[r], d[q]);
            }
            block_sums<8>(d, min(8, j - b0), red + turn * 8 * 16, h + b0, l);
        }
        lds_barrier();
        for (int b = 0; b < j; ++b)
#pragma unroll
            for (int r = 0; r < RM; ++r)
                if (r < a.rounds) w[r] = fma(-h[b], V[(int64_t)b * P + base + r * 64], w[r]);
        lds_barrier();
    }
    part = 0.0;
#pragma unroll
    for (int r = 0; r < RM; ++r) part = fma(w[r], w[r], part);
    const double after = block_sum(part, red1 + 16, l);
    const bool keep = grows(after, before);
    const double norm = sqrt(after);
#pragma unroll
    for (int r = 0; r < RM; ++r)
        if (r < a.rounds) {
            a.W[(int64_t)c * P + base + r * 64] = w[r];
            if (commit) a.V[((int64_t)c * a.kb + j) * P + base + r * 64] = keep ? w[r] / norm : 0.0;
        }
    if (threadIdx.x == 0) {
        ww[c] = after;
        ww0[c] = before;
        if (commit && ke[c] == j && keep) ke[c] = j + 1;
    }
}

__global__ void __launch_bounds__(1024) k_rchip_commit(RChip a, int32_t j, const double *ww, const double *ww0,
                                                       int32_t *ke) {
    const int c = blockIdx.x, P = a.positions;
    const bool keep = grows(ww[c], ww0[c]);
    const double norm = sqrt(ww[c]);
    for (int p = threadIdx.x; p < P; p += blockDim.x)
        a.V[((int64_t)c * a.kb + j) * P + p] = keep ? a.W[(int64_t)c * P + p] / norm : 0.0;
    if (threadIdx.x == 0 && ke[c] == j && keep) ke[c] = j + 1;
}

template <typename F, typename... Args>
hipError_t go(F f, const RChip &a, size_t lds, hipStream_t s, Args... args) {
    if (lds > kResidentLds || a.rounds > RM || a.waves < 1 || a.waves > 16) return hipErrorInvalidValue;
    const hipError_t e =
        hipFuncSetAttribute((const void *)f, hipFuncAttributeMaxDynamicSharedMemorySize, (int)kResidentLds);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(f, dim3(a.cols), dim3(64 * a.waves), lds, s, a, args...);
    return hipGetLastError();
}

}  // namespace

hipError_t launch_rchip_start(const RChip &a, const double *W0, int32_t mp, const double *norm2, hipStream_t s) {
    return go(k_rchip_start, a, 0, s, W0, mp, norm2);
}

hipError_t launch_rchip_project(const RChip &a, int32_t j, double *H, hipStream_t s) {
    const size_t lds = ((size_t)a.positions + 1 + 2 * 8 * 16 + 64) * 8;
    return a.unit ? go(k_rchip_project<true>, a, lds, s, j, H) : go(k_rchip_project<false>, a, lds, s, j, H);
}

hipError_t launch_rchip_solve(const RChip &a, const double *xi, double tol2, int32_t cg_max, int32_t *iters,
                              int64_t *apps, hipStream_t s) {
    // the matrix's words stay in LDS through the iterations where they fit
    const size_t base = ((size_t)a.positions + 1 + 32) * 8, words = (size_t)a.word_rows * 256;
    const bool in = base + words <= kResidentLds;
    const size_t lds = base + (in ? words : 0);
    if (a.unit)
        return in ? go(k_rchip_solve<true, true>, a, lds, s, xi, tol2, cg_max, iters, apps)
                  : go(k_rchip_solve<true, false>, a, lds, s, xi, tol2, cg_max, iters, apps);
    return in ? go(k_rchip_solve<false, true>, a, lds, s, xi, tol2, cg_max, iters, apps)
              : go(k_rchip_solve<false, false>, a, lds, s, xi, tol2, cg_max, iters, apps);
}

hipError_t launch_rchip_orthogonalize(const RChip &a, int32_t j, bool from_u, bool commit, double *ww, double *ww0,
                                      int32_t *ke, hipStream_t s) {
    const size_t lds = (size_t)(2 * 8 * 16 + 64 + 32) * 8;
    return go(k_rchip_orthogonalize, a, lds, s, j, (int32_t)from_u, (int32_t)commit, ww, ww0, ke);
}

hipError_t launch_rchip_commit(const RChip &a, int32_t j, const double *ww, const double *ww0, int32_t *ke,
                               hipStream_t s) {
    return go(k_rchip_commit, a, 0, s, j, ww, ww0, ke);
}

}  // namespace vne
