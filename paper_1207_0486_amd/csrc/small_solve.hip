// A whole FP64 point-Jacobi solve of a small operator in one launch of one
// workgroup: statistics of b, true residuals, the recurrence and its restarts,
// the pure-Neumann normalisation.
//
// The smallest solves are all latency.  As separate launches the 16x16x4 box
// (1,445 rows, 75 iterations) took 437 us, 308 of them in the iterations
// (values read from LDS beside p, sixteen wavefronts) and the rest in about
// twenty one-off launches and four host reads.  Here the matrix stays in
// registers (a thread keeps the diagonal and both triangles of its rows; eight
// wavefronts, so that 256 registers are there for it), p lives in LDS with
// zeros around it, a row's fifteen reads of p are issued while the row before
// is summed, and a sum over the workgroup costs one barrier.  Measured: the box
// 437 -> 157 us; an iteration 1.7 us up to 1,536 rows (3.1 to 4.3 before), 3.4
// against 4.7 at 2,048 and 7.1 against 8.1 at 2,560, the largest taken.
//
// Solves that the caller advances by a number of iterations (batch sessions)
// keep r and p in their workspace and the rest in SmallState between launches:
// the arithmetic does not depend on where a launch ends.
#include <cmath>

#include "device_util.h"
#include "kernels.h"

namespace hns {
namespace {

constexpr int kST = kSmallSolveBlock;
constexpr int kSW = kST / 64;
constexpr int kSM = kSmallSolveDiag;

struct SmallArgs {
    int n, omax;
    int32_t off[kSM];
    const double *dia, *dinv, *b, *lumped;
    double lumped_sum;
    double *x, *r, *p;
    const uint8_t *bc;
    int bit, singular;
    double tol2;
    int max_iter, count, resume;
    SmallState *st;
};

// Sums over the workgroup, in every thread, bit-identical (two sets of slots
// take turns: a set is written again after the barrier of the sum between)
template <int NV>
__device__ __forceinline__ void all_sum(double (&v)[NV], double (*red)[kSW][3], int &turn)
{
    const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
#pragma unroll
    for (int k = 0; k < NV; ++k) v[k] = wave_sum(v[k]);
    if (lane == 0) {
#pragma unroll
        for (int k = 0; k < NV; ++k) red[turn][wid][k] = v[k];
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < NV; ++k) {
        v[k] = 0.0;
#pragma unroll
        for (int w = 0; w < kSW; ++w) v[k] += red[turn][w][k];
    }
    turn ^= 1;
}

// AHEAD: a row's reads of p are issued while the row before is summed (where the
// registers allow it: up to three rows per thread).
template <int ROWS, bool AHEAD>
__global__ __launch_bounds__(kST) __attribute__((amdgpu_waves_per_eu(2, 2)))
void k_small_solve(SmallArgs a)
{
    extern __shared__ double small_p[];   // omax zeros, the n values, omax zeros
    __shared__ double red[2][kSW][3];
    int turn = 0;
    const int n = a.n;
    double *sp = small_p + a.omax;
    for (int i = threadIdx.x; i < n + 2 * a.omax; i += kST) small_p[i] = 0.0;
    double dg[ROWS], up[ROWS][kSM], lo[ROWS][kSM], dv[ROWS], xv[ROWS], rv[ROWS],
        qv[ROWS];
    uint32_t live = 0, fixed = 0;
    double mean_b = 0.0;
    SmallState s{};
    if (a.resume) s = *a.st;
    __syncthreads();   // zeros before the values below
#pragma unroll
    for (int j = 0; j < ROWS; ++j) {
        const int i = threadIdx.x + j * kST;
        const bool ex = i < n;
        if (ex) live |= 1u << j;
        if (!ex || is_dirichlet(a.bc, a.bit, i)) fixed |= 1u << j;
        const int ic = ex ? i : 0;
        dg[j] = ex ? a.dia[ic] : 0.0;
        dv[j] = ex ? a.dinv[ic] : 0.0;
        xv[j] = ex && !((fixed >> j) & 1u) ? a.x[ic] : 0.0;
        rv[j] = 0.0;
#pragma unroll
        for (int k = 0; k < kSM; ++k) {
            const int o = a.off[k];
            const double *u = a.dia + (int64_t)(k + 1) * n;
            up[j][k] = ex && i + o < n ? u[ic] : 0.0;
            lo[j][k] = ex && i >= o ? u[ic - o] : 0.0;
        }
        __builtin_amdgcn_sched_barrier(0);   // a row's loads at a time: addresses take registers
    }
    // b is read where it is needed (twice in most solves), not kept
    auto load_b = [&](int j) {
        return (fixed >> j) & 1u ? 0.0 : a.b[fresh(threadIdx.x) + j * kST];
    };
    // q = mask(A v) for the vector v in sp
    auto product = [&]() {
        constexpr int B = AHEAD ? 2 : 1;
        double c[B], pu[B][kSM], pl[B][kSM];
        const int t = fresh(threadIdx.x);
        auto gather = [&](int j, int to) {
            const int i = t + j * kST, at = i < n ? i : 0;
            c[to] = sp[at];
#pragma unroll
            for (int k = 0; k < kSM; ++k) {
                pu[to][k] = sp[at + a.off[k]];
                pl[to][k] = sp[at - a.off[k]];
            }
        };
        if (AHEAD) gather(0, 0);
#pragma unroll
        for (int j = 0; j < ROWS; ++j) {
            if (!AHEAD)
                gather(j, 0);
            else if (j + 1 < ROWS)
                gather(j + 1, (j + 1) % B);
            __builtin_amdgcn_sched_barrier(0);
            double sum = dg[j] * c[j % B];
#pragma unroll
            for (int k = 0; k < kSM; ++k) {
                sum += up[j][k] * pu[j % B][k];
                sum += lo[j][k] * pl[j % B][k];
            }
            qv[j] = (fixed >> j) & 1u ? 0.0 : sum;
        }
    };
    auto put = [&](const double (&v)[ROWS]) {   // v into sp, whose readers are done
        __syncthreads();
#pragma unroll
        for (int j = 0; j < ROWS; ++j)
            if ((live >> j) & 1u) sp[fresh(threadIdx.x) + j * kST] = v[j];
        __syncthreads();
    };
    // r = b - A x (projected in the pure-Neumann case), |b|^2 and |r|^2
    auto true_residual = [&](double &bb, double &rr) {
        put(xv);
        product();
        double v[2] = {0.0, 0.0};
#pragma unroll
        for (int j = 0; j < ROWS; ++j) {
            const bool in = !((fixed >> j) & 1u);
            const double bj = in ? load_b(j) - mean_b : 0.0;
            rv[j] = in ? bj - qv[j] : 0.0;
            v[0] += rv[j];
            v[1] += bj * bj;
        }
        all_sum<2>(v, red, turn);
        bb = v[1];
        const double mean = a.singular ? v[0] / (double)n : 0.0;
        double w[1] = {0.0};
#pragma unroll
        for (int j = 0; j < ROWS; ++j) {
            if ((live >> j) & 1u) rv[j] -= mean;
            w[0] += rv[j] * rv[j];
        }
        all_sum<1>(w, red, turn);
        rr = w[0];
    };
    int stop = 0;
    // p = z = D^-1 r, rho = r^T z
    auto start = [&]() {
        double v[1] = {0.0};
        __syncthreads();
#pragma unroll
        for (int j = 0; j < ROWS; ++j) {
            const double z = dv[j] * rv[j];
            if ((live >> j) & 1u) sp[fresh(threadIdx.x) + j * kST] = z;
            v[0] += rv[j] * z;
        }
        all_sum<1>(v, red, turn);
        s.rho = v[0];
        stop = isfinite(s.rho) ? 0 : 2;
    };

    if (!a.resume) {
        double v[2] = {0.0, 0.0};
#pragma unroll
        for (int j = 0; j < ROWS; ++j) {
            const double bj = load_b(j);
            if (isfinite(bj))
                v[0] += bj;
            else
                v[1] += 1.0;
        }
        all_sum<2>(v, red, turn);
        s.nonfinite = v[1];
        s.mean_b = a.singular ? v[0] / (double)n : 0.0;
        mean_b = s.mean_b;
        s.rr_best = INFINITY;
        if (s.nonfinite > 0.0) {
            s.phase = SmallState::kBadRhs;
        } else {
            true_residual(s.bb, s.rr_true);
            if (!(s.bb > 0.0)) {
                s.phase = SmallState::kZero;
#pragma unroll
                for (int j = 0; j < ROWS; ++j) xv[j] = 0.0;
            } else if (!(s.rr_true > a.tol2 * s.bb)) {
                s.phase = SmallState::kDone;
            } else {
                start();
            }
        }
    } else {
        mean_b = s.mean_b;
#pragma unroll
        for (int j = 0; j < ROWS; ++j) {
            const int i = threadIdx.x + j * kST;
            if (i < n) {
                rv[j] = a.r[i];
                sp[i] = a.p[i];
            }
        }
        __syncthreads();
    }

    int left = a.count;
    while (s.phase == SmallState::kRunning) {
        const double limit = a.tol2 * s.bb;
        while (stop == 0 && left > 0 && s.iter < a.max_iter) {
            product();
            double v1[1] = {0.0};
#pragma unroll
            for (int j = 0; j < ROWS; ++j)
                if ((live >> j) & 1u) v1[0] += sp[fresh(threadIdx.x) + j * kST] * qv[j];
            all_sum<1>(v1, red, turn);
            s.gamma = v1[0];
            if (!(s.gamma > 0.0) || !isfinite(s.gamma)) {
                stop = 2;
                break;
            }
            const double alpha = s.rho / s.gamma;
            double v2[2] = {0.0, 0.0};
#pragma unroll
            for (int j = 0; j < ROWS; ++j) {
                rv[j] = rv[j] - alpha * qv[j];
                v2[0] += rv[j] * (dv[j] * rv[j]);
                v2[1] += rv[j] * rv[j];
            }
            all_sum<2>(v2, red, turn);
            const bool bad = !isfinite(v2[0]) || !isfinite(v2[1]);
            const bool conv = !bad && v2[1] <= limit;
            const double beta = v2[0] / s.rho;
#pragma unroll
            for (int j = 0; j < ROWS; ++j)
                if ((live >> j) & 1u) {
                    const int i = fresh(threadIdx.x) + j * kST;
                    const double pi = sp[i];
                    xv[j] = xv[j] + alpha * pi;
                    sp[i] = dv[j] * rv[j] + beta * pi;
                }
            s.rho = v2[0];
            ++s.iter;
            --left;
            stop = bad ? 2 : conv ? 1 : 0;
            __syncthreads();
        }
        if (stop == 2) {
            s.phase = SmallState::kBreakdown;
            break;
        }
        if (stop == 0 && s.iter < a.max_iter) break;   // this launch's iterations are done
        double bb;
        true_residual(bb, s.rr_true);
        if (s.rr_true <= limit) {
            s.phase = SmallState::kDone;
        } else if (stop != 1 || s.iter >= a.max_iter) {
            s.phase = SmallState::kCapped;
        } else {
            // the rounding floor: three failed checks in a row that do not
            // halve the smallest true residual seen at a check end the solve
            s.floor_checks = s.rr_true > 0.25 * s.rr_best ? s.floor_checks + 1 : 0;
            s.rr_best = fmin(s.rr_best, s.rr_true);
            if (s.floor_checks >= 3)
                s.phase = SmallState::kFloor;
            else
                start();
        }
    }

    if (s.phase == SmallState::kBadRhs) {
        if (threadIdx.x == 0) *a.st = s;
        return;
    }
    if (s.phase == SmallState::kRunning) {
#pragma unroll
        for (int j = 0; j < ROWS; ++j) {
            const int i = threadIdx.x + j * kST;
            if (i < n) {
                a.r[i] = rv[j];
                a.p[i] = sp[i];
            }
        }
    } else if (s.phase != SmallState::kBreakdown && a.singular) {
        // zero mass-weighted mean
        double v[1] = {0.0};
#pragma unroll
        for (int j = 0; j < ROWS; ++j)
            if ((live >> j) & 1u) v[0] += a.lumped[threadIdx.x + j * kST] * xv[j];
        all_sum<1>(v, red, turn);
        const double shift = v[0] / a.lumped_sum;
#pragma unroll
        for (int j = 0; j < ROWS; ++j) xv[j] -= shift;
    }
#pragma unroll
    for (int j = 0; j < ROWS; ++j) {
        const int i = threadIdx.x + j * kST;
        if (i < n) a.x[i] = xv[j];
    }
    if (threadIdx.x == 0) *a.st = s;
}

}  // namespace

// Rows a thread keeps at most (five rows of fifteen values, and x, r, q, b,
// D^-1 of each, take the 256 registers of a lane)
static_assert(kSmallSolveRows <= 5 * kSmallSolveBlock, "instances below");

hns_status launch_small_solve(const DevMatrix &A, const double *dinv, const double *b, double *x,
                              double *r, double *p, const uint8_t *bc, int bit, bool singular,
                              const double *lumped, double lumped_sum, double tol, int max_iter,
                              int count, bool resume, SmallState *st, hipStream_t s)
{
    if (!small_solve_fits(A) || count < 0) {
        set_error("launch_small_solve: unsupported configuration");
        return HNS_ERR_INVALID;
    }
    SmallArgs a{};
    a.n = (int)A.n;
    a.omax = A.off[kSM - 1];
    for (int k = 0; k < kSM; ++k) a.off[k] = A.off[k];
    a.dia = A.dia;
    a.dinv = dinv;
    a.b = b;
    a.lumped = lumped;
    a.lumped_sum = lumped_sum;
    a.x = x;
    a.r = r;
    a.p = p;
    a.bc = bit < 0 ? nullptr : bc;
    a.bit = bit < 0 ? 0 : bit;
    a.singular = singular;
    a.tol2 = tol * tol;
    a.max_iter = max_iter;
    a.count = count;
    a.resume = resume;
    a.st = st;
    const size_t shm = (size_t)(a.n + 2 * a.omax) * sizeof(double);
    switch ((a.n + kST - 1) / kST) {
    case 1: k_small_solve<1, false><<<1, kST, shm, s>>>(a); break;
    case 2: k_small_solve<2, true><<<1, kST, shm, s>>>(a); break;
    case 3: k_small_solve<3, true><<<1, kST, shm, s>>>(a); break;
    case 4: k_small_solve<4, false><<<1, kST, shm, s>>>(a); break;
    default: k_small_solve<5, false><<<1, kST, shm, s>>>(a); break;
    }
    HNS_TRY_HIP(hipGetLastError());
    return HNS_OK;
}

}  // namespace hns
