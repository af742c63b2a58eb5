// Right-hand sides and corrections of one projection time step (Sec. 3,
// weak forms of Sec. 4 discretised as in Sec. 5), built from the auxiliary
// forms kept on a HNS_STEP_AUX operator.  All work runs in the kernels
// below and the library's CSR SpMV.
#include <algorithm>
#include <cmath>

#include "device_util.h"
#include "kernels.h"

namespace hns {
namespace {

#define GRID_STRIDE(i, n)                                                   \
    for (int64_t i = blockIdx.x * (int64_t)kBlock + threadIdx.x; i < (n); \
         i += (int64_t)gridDim.x * kBlock)

__device__ __forceinline__ bool dirichlet(const uint8_t *bc, int bit, int64_t i)
{
    return bc != nullptr && ((bc[i] >> bit) & 1u);
}

// Three consecutive doubles at an 8-byte aligned place
struct Three {
    double v[3];
};

__device__ __forceinline__ Three load3(const double *p)
{
    Three t;
    __builtin_memcpy(&t, p, sizeof(t));
    return t;
}

__device__ __forceinline__ void store3(double *p, const Three &t)
{
    __builtin_memcpy(p, &t, sizeof(t));
}

// y += a x
__global__ __launch_bounds__(kBlock) void k_axpy(int64_t n, double *__restrict__ y, double a,
                                                 const double *__restrict__ x)
{
    GRID_STRIDE(i, n) y[i] += a * x[i];
}

// y = a .* b
__global__ __launch_bounds__(kBlock) void k_hadamard(int64_t n, double *__restrict__ y,
                                                     const double *__restrict__ a,
                                                     const double *__restrict__ b)
{
    GRID_STRIDE(i, n) y[i] = a[i] * b[i];
}

// y = a x
__global__ __launch_bounds__(kBlock) void k_scale(int64_t n, double *__restrict__ y, double a,
                                                  const double *__restrict__ x)
{
    GRID_STRIDE(i, n) y[i] = a * x[i];
}

__global__ __launch_bounds__(kBlock) void k_mask(int64_t n, double *__restrict__ y,
                                                 const uint8_t *__restrict__ bc, int bit)
{
    GRID_STRIDE(i, n)
    if (dirichlet(bc, bit, i)) y[i] = 0.0;
}

// u = mask(ut - dt * g / m_L)
__global__ __launch_bounds__(kBlock) void k_correct_lumped(int64_t n, double *__restrict__ u,
                                                           const double *__restrict__ ut,
                                                           const double *__restrict__ g,
                                                           const double *__restrict__ mL, double dt,
                                                           const uint8_t *__restrict__ bc,
                                                           int bit)
{
    GRID_STRIDE(i, n) u[i] = dirichlet(bc, bit, i) ? 0.0 : ut[i] - dt * g[i] / mL[i];
}

// One row per thread, each XCD on a contiguous eighth of the rows (row i - o of
// every array was read a little earlier by the same XCD: 349K rows, prediction
// 52 -> 43 us, pressure 31 -> 23 us (5.9 TB/s) against a grid-stride loop).
__device__ __forceinline__ int64_t form_row()
{
    return (int64_t)xcd_block(blockIdx.x, gridDim.x) * kBlock + threadIdx.x;
}

int form_grid(int64_t n)
{
    const int64_t g = (n + kBlock - 1) / kBlock;
    return (int)(g >= 8 ? (g + 7) / 8 * 8 : g);
}

// Velocity components of a node side by side: a vertex of the advection term is
// then two runs of 24 bytes instead of three and three 8-byte gathers
__global__ __launch_bounds__(kBlock) void k_interleave(int64_t n, const double *__restrict__ u,
                                                       double *__restrict__ out)
{
    GRID_STRIDE(i, n)
    {
        Three v;
#pragma unroll
        for (int c = 0; c < 3; ++c) v.v[c] = u[c * n + i];
        store3(out + 3 * i, v);
    }
}

// out_c[a] = int ((u . grad) u_c) phi_a over the tetrahedra around node a,
// for c = 1..3 (explicit advection of the velocity prediction).  On a
// tetrahedron with basis gradients g_b the gradient of u_c is the constant
// G_c = sum_b u_c(b) g_b; (u . grad) u_c = sum_b phi_b s_b with
// s_b = u(b) . G_c, and int phi_a phi_b = vol/20 (1 + delta_ab) gives the
// node's share vol/20 (sum_b u(b) + u(a)) . G_c.  With the three other
// vertices k of the positively oriented tetrahedron seen from a, edges e_k and
// C_1 = e_2 x e_3 (cyclic), D = 6 vol, G_c is sum_k (u_c(k) - u_c(a)) C_k / D,
// so D cancels: the share is (sum_b u(b) + u(a)) . sum_k (u_c(k) - u_c(a)) C_k
// / 120, without a division.
// kAdvLanes lanes per node take its tetrahedra in turn (ascending order) and
// are summed in lane order: deterministic, no atomics; the geometry is
// recomputed from the coordinates.  Bound by the gathers (a tetrahedron is
// visited by its four vertices): 349K nodes, one lane per node and the
// gradients formed first 350 us; this form 93 us with 4 or 8 lanes.
constexpr int kAdvLanes = 4;

__global__ __launch_bounds__(kBlock) void k_advection(int64_t n, const double *__restrict__ xyz,
                                                      const int32_t *__restrict__ tets,
                                                      const int64_t *__restrict__ ptr,
                                                      const int32_t *__restrict__ itet,
                                                      const int8_t *__restrict__ iloc,
                                                      const double *__restrict__ u3,
                                                      double *__restrict__ out)
{
    const int part = threadIdx.x % kAdvLanes;
    const int64_t a = form_row() / kAdvLanes;   // a workgroup: consecutive nodes
    {
        double acc[3] = {0.0, 0.0, 0.0};
        if (a < n) {
            const Three xa = load3(xyz + 3 * a), ua = load3(u3 + 3 * a);
            const int64_t s1 = ptr[a + 1];
            for (int64_t s = ptr[a] + part; s < s1; s += kAdvLanes) {
                const int4 t = *reinterpret_cast<const int4 *>(tets + 4 * (int64_t)itet[s]);
                // the others in an order that keeps the orientation (an even
                // permutation with a in front)
                const int la = iloc[s];
                const int32_t o1 = la == 0 ? t.y : t.x;
                const int32_t o2 = la == 0 || la == 3 ? t.z : la == 2 ? t.y : t.w;
                const int32_t o3 = la == 0 || la == 2 ? t.w : la == 1 ? t.z : t.y;
                const int32_t o[3] = {o1, o2, o3};
                double e[3][3], d[3][3], su[3];
#pragma unroll
                for (int c = 0; c < 3; ++c) su[c] = 2.0 * ua.v[c];
#pragma unroll
                for (int k = 0; k < 3; ++k) {
                    const Three x = load3(xyz + 3 * (int64_t)o[k]), w = load3(u3 + 3 * (int64_t)o[k]);
#pragma unroll
                    for (int c = 0; c < 3; ++c) {
                        e[k][c] = x.v[c] - xa.v[c];
                        d[k][c] = w.v[c] - ua.v[c];
                        su[c] += w.v[c];
                    }
                }
                // su . C_k, then the node's share
                double f[3];
#pragma unroll
                for (int k = 0; k < 3; ++k) {
                    const double *p = e[(k + 1) % 3], *q = e[(k + 2) % 3];
                    f[k] = su[0] * (p[1] * q[2] - p[2] * q[1]) +
                           su[1] * (p[2] * q[0] - p[0] * q[2]) +
                           su[2] * (p[0] * q[1] - p[1] * q[0]);
                }
#pragma unroll
                for (int c = 0; c < 3; ++c)
                    acc[c] += f[0] * d[0][c] + f[1] * d[1][c] + f[2] * d[2][c];
            }
        }
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            double v = acc[c];
#pragma unroll
            for (int d = 1; d < kAdvLanes; d *= 2) v += __shfl_xor(v, d, kAdvLanes);
            acc[c] = v;
        }
        if (a < n && part < 3)
            out[part * n + a] = (part == 0 ? acc[0] : part == 1 ? acc[1] : acc[2]) / 120.0;
    }
}

// u = mask(x)  (copy with the Dirichlet entries of bit set to 0)
__global__ __launch_bounds__(kBlock) void k_copy_masked(int64_t n, double *__restrict__ y,
                                                        const double *__restrict__ x,
                                                        const uint8_t *__restrict__ bc, int bit)
{
    GRID_STRIDE(i, n) y[i] = dirichlet(bc, bit, i) ? 0.0 : x[i];
}

// ---------------------------------------------------------------------------
// The forms of a step in diagonal storage, all components in one pass.  M keeps
// its symmetric diagonals (M_0, then the upper ones), B_c three arrays per
// offset o: U(i) = B(i, i + o) and L(i) = B(i + o, i) (and the diagonal), so
// row i of B reads U(i) and L(i - o) and row i of B^T the same with U and L
// exchanged.  Every array is read along the rows, no indices: 8 (2 m + 1) bytes
// per row and component against 12 per entry of compressed rows, and what a
// separate product, scaling and addition wrote and read again stays in
// registers.  Bound by memory: the 45 arrays of B are 3/4 of the bytes.
// An absent coupling takes no part (a non-finite value at an unconnected node
// stays where it is): in M it is a stored 0, where a present one is positive; in
// B, whose present couplings may be exactly 0 (two tetrahedra cancel on uniform
// meshes), it is kNoCoupling, and a present 0 is multiplied like any other.
// ---------------------------------------------------------------------------
struct FormOffsets {
    int32_t o[kMaxDiag];
};

struct FormArgs {
    int64_t n;
    int m;                // upper diagonals
    FormOffsets offs;
    const double *M;      // (m + 1) n
    const double *B;      // 3 (2 m + 1) n: per component the diagonal, U's, L's
    const uint8_t *bc;
};

__device__ __forceinline__ double times(double a, double x) { return a != 0.0 ? a * x : 0.0; }

// the same for an entry of B
__device__ __forceinline__ double div_times(double a, double x)
{
    return __double_as_longlong(a) != __double_as_longlong(kNoCoupling) ? a * x : 0.0;
}

// (M v_c)(i) for the NC vectors v + c n
template <int NC>
__device__ __forceinline__ void mass_row(const FormArgs &f, int64_t i, const double *v,
                                         double (&acc)[3])
{
    const int m = f.m;
    const int64_t n = f.n;
    const double d = f.M[i];
#pragma unroll
    for (int c = 0; c < NC; ++c) acc[c] = d * v[c * n + i];
#pragma unroll 2
    for (int k = 0; k < m; ++k) {
        const int64_t o = f.offs.o[k], iu = i + o < n ? i + o : n - 1, il = i >= o ? i - o : 0;
        const double *A = f.M + (k + 1) * n;
        const double au = i + o < n ? A[i] : 0.0, al = i >= o ? A[il] : 0.0;
#pragma unroll
        for (int c = 0; c < NC; ++c) acc[c] += times(au, v[c * n + iu]) + times(al, v[c * n + il]);
    }
}

// acc[c] = (B_c x_c)(i), or (B_c^T x_c)(i) with TR; SAME: one x for the three
template <bool TR, bool SAME>
__device__ __forceinline__ void div_row(const FormArgs &f, int64_t i, const double *x,
                                        double (&acc)[3])
{
    const int m = f.m;
    const int64_t n = f.n, per = (int64_t)(2 * m + 1) * n;
#pragma unroll
    for (int c = 0; c < 3; ++c) acc[c] = div_times(f.B[c * per + i], x[(SAME ? 0 : c * n) + i]);
#pragma unroll 2
    for (int k = 0; k < m; ++k) {
        const int64_t o = f.offs.o[k], iu = i + o < n ? i + o : n - 1, il = i >= o ? i - o : 0;
        const int ku = TR ? 1 + m + k : 1 + k, kl = TR ? 1 + k : 1 + m + k;
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            const double *Bc = f.B + c * per;
            const double au = i + o < n ? Bc[ku * n + i] : kNoCoupling;
            const double al = i >= o ? Bc[kl * n + il] : kNoCoupling;
            const double *xc = x + (SAME ? 0 : c * n);
            acc[c] += div_times(au, xc[iu]) + div_times(al, xc[il]);
        }
    }
}

// v_c = a1 u_c + a2 u'_c and the Coriolis exchange +-tau f u_o: what M multiplies
// in the prediction right-hand side (one product per component instead of three)
__global__ __launch_bounds__(kBlock) void k_mass_input(int64_t n, double tau, double a1,
                                                       const double *__restrict__ u, double a2,
                                                       const double *__restrict__ up,
                                                       const double *__restrict__ f,
                                                       double *__restrict__ v)
{
    GRID_STRIDE(i, n)
    {
        const double u1 = u[i], u2 = u[n + i], u3 = u[2 * n + i];
        double v1 = a1 * u1, v2 = a1 * u2, v3 = a1 * u3;
        if (a2 != 0.0) {
            v1 += a2 * up[i];
            v2 += a2 * up[n + i];
            v3 += a2 * up[2 * n + i];
        }
        if (f) {
            const double tf = tau * f[i];
            v1 += tf * u2;
            v2 -= tf * u1;
        }
        v[i] = v1;
        v[n + i] = v2;
        v[2 * n + i] = v3;
    }
}

// b_c = M v_c + tau (M_s theta_c - adv_c + B_c^T p), 0 on the Dirichlet sets
__global__ __launch_bounds__(kBlock) void k_velocity_rhs(
    FormArgs f, double tau, const double *__restrict__ v, const double *__restrict__ p,
    const int32_t *__restrict__ sptr, const int32_t *__restrict__ scol,
    const double *__restrict__ sval, const double *__restrict__ theta, const double *adv,
    double *b)
{
    const int64_t n = f.n;
    const int64_t i = form_row();
    if (i < n)
    {
        double acc[3], g[3] = {0.0, 0.0, 0.0};
        mass_row<3>(f, i, v, acc);
        if (p) div_row<true, true>(f, i, p, g);
        if (theta) {
            double t0 = 0.0, t1 = 0.0;   // rows of surface nodes only
            for (int32_t k = sptr[i]; k < sptr[i + 1]; ++k) {
                t0 += sval[k] * theta[scol[k]];
                t1 += sval[k] * theta[n + scol[k]];
            }
            g[0] += t0;
            g[1] += t1;
        }
        const unsigned bits = f.bc ? f.bc[i] : 0u;
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            if (adv) g[c] -= adv[c * n + i];
            b[c * n + i] = (bits >> c) & 1u ? 0.0 : acc[c] + tau * g[c];
        }
    }
}

// b = scale sum_c B_c ut_c
__global__ __launch_bounds__(kBlock) void k_pressure_rhs(FormArgs f, double scale,
                                                         const double *__restrict__ ut,
                                                         double *__restrict__ b)
{
    const int64_t i = form_row();
    if (i < f.n)
    {
        double g[3];
        div_row<false, false>(f, i, ut, g);
        b[i] = scale * (g[0] + g[1] + g[2]);
    }
}

// p += q; r_c = M ut_c - tau B_c q, 0 on the Dirichlet sets
__global__ __launch_bounds__(kBlock) void k_correct_rhs(FormArgs f, double tau,
                                                        const double *__restrict__ ut,
                                                        const double *__restrict__ q, double *p,
                                                        double *__restrict__ r)
{
    const int64_t n = f.n;
    const int64_t i = form_row();
    if (i < n)
    {
        double acc[3], g[3];
        mass_row<3>(f, i, ut, acc);
        div_row<false, true>(f, i, q, g);
        const unsigned bits = f.bc ? f.bc[i] : 0u;
        if (p) p[i] += q[i];
#pragma unroll
        for (int c = 0; c < 3; ++c) r[c * n + i] = (bits >> c) & 1u ? 0.0 : acc[c] - tau * g[c];
    }
}

// p += q; u_c = ut_c - dt (B_c q) / m_L, 0 on the Dirichlet sets (u may be ut)
__global__ __launch_bounds__(kBlock) void k_correct(FormArgs f, double dt, const double *ut,
                                                    const double *__restrict__ q, double *p,
                                                    const double *__restrict__ mL, double *u)
{
    const int64_t n = f.n;
    const int64_t i = form_row();
    if (i < n)
    {
        double g[3];
        div_row<false, true>(f, i, q, g);
        const unsigned bits = f.bc ? f.bc[i] : 0u;
        if (p) p[i] += q[i];
#pragma unroll
        for (int c = 0; c < 3; ++c)
            u[c * n + i] = (bits >> c) & 1u ? 0.0 : ut[c * n + i] - dt * g[c] / mL[i];
    }
}

// y = B_c x or B_c^T x for one component
template <bool TR>
__global__ __launch_bounds__(kBlock) void k_div_apply(FormArgs f, const double *__restrict__ x,
                                                      double *__restrict__ y)
{
    const int64_t n = f.n;
    GRID_STRIDE(i, n)
    {
        double s = div_times(f.B[i], x[i]);
        for (int k = 0; k < f.m; ++k) {
            const int64_t o = f.offs.o[k];
            const double *U = f.B + (TR ? 1 + f.m + k : 1 + k) * n;
            const double *L = f.B + (TR ? 1 + k : 1 + f.m + k) * n;
            if (i + o < n) s += div_times(U[i], x[i + o]);
            if (i >= o) s += div_times(L[i - o], x[i - o]);
        }
        y[i] = s;
    }
}

FormArgs form_args(const hns_operator *op)
{
    FormArgs f{};
    f.n = op->n;
    f.m = op->M.ndiag;
    for (int k = 0; k < f.m; ++k) f.offs.o[k] = op->M.off[k];
    f.M = op->M.dia;
    f.B = op->Bdia;
    f.bc = op->bc;
    return f;
}

bool overlaps(const double *a, int64_t na, const double *b, int64_t nb)
{
    return a && b && a < b + nb && b < a + na;
}

// The corrections add q to p before they read u~ and write the result; in one
// launch that order holds only where p shares memory with none of them
bool p_alone(int64_t n, const double *p, const double *q, const double *ut, const double *out)
{
    return !overlaps(p, n, q, n) && !overlaps(p, n, ut, 3 * n) && !overlaps(p, n, out, 3 * n);
}

hns_status check(const char *what)
{
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) {
        set_error("launch of %s failed: %s", what, hipGetErrorString(e));
        return HNS_ERR_HIP;
    }
    return HNS_OK;
}

hns_status need_aux(const hns_operator *op)
{
    if (!op) {
        set_error("null operator");
        return HNS_ERR_INVALID;
    }
    if (!op->has_aux) {
        set_error("the operator was not assembled with HNS_STEP_AUX");
        return HNS_ERR_INVALID;
    }
    return HNS_OK;
}

// y = B_c x (or B_c^T x) as a launch of its own
hns_status apply_div(const hns_operator *op, int c, bool transposed, const double *x, double *y,
                     hipStream_t s)
{
    if (!op->Bdia)
        return launch_spmv_plain(transposed ? op->Bt[c] : op->B[c], false, x, y, nullptr, -1, s);
    FormArgs f = form_args(op);
    f.B += (int64_t)c * (2 * f.m + 1) * f.n;
    auto k = transposed ? k_div_apply<true> : k_div_apply<false>;
    k<<<stream_grid(f.n), kBlock, 0, s>>>(f, x, y);
    return check("divergence form");
}

}  // namespace
}  // namespace hns

using namespace hns;

extern "C" {

hns_status hns_apply_aux(hns_operator *op, int which, const double *x_dev, double *y_dev,
                         void *stream)
{
    HNS_TRY(need_aux(op));
    if (!x_dev || !y_dev || which < 0 || which > 7) {
        set_error("hns_apply_aux: bad arguments");
        return HNS_ERR_INVALID;
    }
    if (which >= 1 && which <= 6) {
        HNS_TRY(apply_div(op, (which - 1) % 3, which > 3, x_dev, y_dev, (hipStream_t)stream));
        HNS_TRY_HIP(hipStreamSynchronize((hipStream_t)stream));
        return HNS_OK;
    }
    const DevMatrix *F = which == 0 ? &op->M : &op->Ms;
    hipStream_t s = (hipStream_t)stream;
    HNS_TRY(launch_spmv_plain(*F, false, x_dev, y_dev, nullptr, -1, s));
    HNS_TRY_HIP(hipStreamSynchronize(s));
    return HNS_OK;
}

static hns_status velocity_rhs(hns_operator *op, double tau, double a1, const double *u_dev,
                               double a2, const double *uprev_dev, const double *p_dev,
                               const double *theta_dev, const double *f_dev,
                               const double *adv_dev, double *b_dev, hipStream_t s);
static hns_status pressure_rhs(hns_operator *op, double scale, const double *ut_dev,
                               double *b_dev, hipStream_t s);

hns_status hns_step_velocity_rhs(hns_operator *op, const double *u_dev, const double *p_dev,
                                 const double *theta_dev, const double *f_dev, double *b_dev,
                                 void *stream)
{
    HNS_TRY(need_aux(op));
    if (!u_dev || !b_dev) {
        set_error("hns_step_velocity_rhs: null velocity or output");
        return HNS_ERR_INVALID;
    }
    return velocity_rhs(op, op->dt, 1.0, u_dev, 0.0, nullptr, p_dev, theta_dev, f_dev, nullptr,
                        b_dev, (hipStream_t)stream);
}

hns_status hns_step_pressure_rhs(hns_operator *op, const double *ut_dev, double *b_dev,
                                 void *stream)
{
    HNS_TRY(need_aux(op));
    if (!ut_dev || !b_dev || !(op->dt != 0.0)) {
        set_error("hns_step_pressure_rhs: null vector or zero time step");
        return HNS_ERR_INVALID;
    }
    return pressure_rhs(op, -1.0 / op->dt, ut_dev, b_dev, (hipStream_t)stream);
}

hns_status hns_step_correct(hns_operator *op, const double *ut_dev, const double *q_dev,
                            double *p_dev, double *u_dev, void *stream)
{
    HNS_TRY(need_aux(op));
    if (!ut_dev || !q_dev || !u_dev) {
        set_error("hns_step_correct: null vector");
        return HNS_ERR_INVALID;
    }
    hipStream_t s = (hipStream_t)stream;
    if (op->Bdia && !overlaps(q_dev, op->n, u_dev, 3 * op->n) &&
        p_alone(op->n, p_dev, q_dev, ut_dev, u_dev)) {
        const FormArgs f = form_args(op);
        k_correct<<<form_grid(f.n), kBlock, 0, s>>>(f, op->dt, ut_dev, q_dev, p_dev, op->lumped, u_dev);
        HNS_TRY(check("correction"));
        HNS_TRY_HIP(hipStreamSynchronize(s));
        return HNS_OK;
    }
    const int64_t n = op->n;
    const int G = stream_grid(n);
    std::lock_guard<std::mutex> scratch(op->step_mutex);
    double *t0 = op->step_tmp;
    if (p_dev) {
        k_axpy<<<G, kBlock, 0, s>>>(n, p_dev, 1.0, q_dev);
        HNS_TRY(check("pressure update"));
    }
    for (int c = 0; c < 3; ++c) {
        HNS_TRY(apply_div(op, c, false, q_dev, t0, s));
        k_correct_lumped<<<G, kBlock, 0, s>>>(n, u_dev + c * n, ut_dev + c * n, t0, op->lumped,
                                              op->dt, op->bc, c);
        HNS_TRY(check("velocity correction"));
    }
    HNS_TRY_HIP(hipStreamSynchronize(s));
    return HNS_OK;
}

hns_status hns_step_advection(hns_operator *op, const double *u_dev, double *out_dev,
                              void *stream)
{
    HNS_TRY(need_aux(op));
    if (!u_dev || !out_dev || u_dev == out_dev) {
        set_error("hns_step_advection: null or aliased vectors");
        return HNS_ERR_INVALID;
    }
    hipStream_t s = (hipStream_t)stream;
    std::lock_guard<std::mutex> scratch(op->step_mutex);
    k_interleave<<<stream_grid(op->n), kBlock, 0, s>>>(op->n, u_dev, op->step_tmp);
    HNS_TRY(check("advection"));
    k_advection<<<form_grid(op->n * kAdvLanes), kBlock, 0, s>>>(
        op->n, op->mesh_xyz, op->mesh_tets, op->inc_ptr, op->inc_tet, op->inc_loc, op->step_tmp,
        out_dev);
    HNS_TRY(check("advection"));
    HNS_TRY_HIP(hipStreamSynchronize(s));
    return HNS_OK;
}

hns_status hns_step_velocity_rhs_bdf(hns_operator *op, double tau, double a1, const double *u_dev,
                                     double a2, const double *uprev_dev, const double *p_dev,
                                     const double *theta_dev, const double *f_dev,
                                     const double *adv_dev, double *b_dev, void *stream)
{
    HNS_TRY(need_aux(op));
    if (!u_dev || !b_dev || (a2 != 0.0 && !uprev_dev) || !std::isfinite(tau) ||
        !std::isfinite(a1) || !std::isfinite(a2)) {
        set_error("hns_step_velocity_rhs_bdf: null vector or non-finite coefficient");
        return HNS_ERR_INVALID;
    }
    return velocity_rhs(op, tau, a1, u_dev, a2, uprev_dev, p_dev, theta_dev, f_dev, adv_dev,
                        b_dev, (hipStream_t)stream);
}

static hns_status velocity_rhs(hns_operator *op, double tau, double a1, const double *u_dev,
                               double a2, const double *uprev_dev, const double *p_dev,
                               const double *theta_dev, const double *f_dev,
                               const double *adv_dev, double *b_dev, hipStream_t s)
{
    const int64_t n = op->n;
    const int G = stream_grid(n);
    std::lock_guard<std::mutex> scratch(op->step_mutex);
    if (op->Bdia && !overlaps(b_dev, 3 * n, p_dev, n) && !overlaps(b_dev, 3 * n, theta_dev, 2 * n)) {
        const FormArgs f = form_args(op);
        double *v = op->step_tmp;
        k_mass_input<<<G, kBlock, 0, s>>>(n, tau, a1, u_dev, a2, uprev_dev, f_dev, v);
        HNS_TRY(check("prediction right-hand side"));
        k_velocity_rhs<<<form_grid(n), kBlock, 0, s>>>(f, tau, v, p_dev, op->Ms.rowptr, op->Ms.col,
                                            op->Ms.val, theta_dev, adv_dev, b_dev);
        HNS_TRY(check("prediction right-hand side"));
        HNS_TRY_HIP(hipStreamSynchronize(s));
        return HNS_OK;
    }
    double *t0 = op->step_tmp, *t1 = op->step_tmp + n;
    for (int c = 0; c < 3; ++c) {
        double *b = b_dev + c * n;
        HNS_TRY(launch_spmv_plain(op->M, false, u_dev + c * n, t0, nullptr, -1, s));
        k_scale<<<G, kBlock, 0, s>>>(n, b, a1, t0);                       // a1 M u_c
        HNS_TRY(check("scale"));
        if (a2 != 0.0) {                                                   // + a2 M u'_c
            HNS_TRY(launch_spmv_plain(op->M, false, uprev_dev + c * n, t0, nullptr, -1, s));
            k_axpy<<<G, kBlock, 0, s>>>(n, b, a2, t0);
            HNS_TRY(check("axpy"));
        }
        if (theta_dev && c < 2) {                                          // + tau M_s theta_c
            HNS_TRY(launch_spmv_plain(op->Ms, false, theta_dev + c * n, t0, nullptr, -1, s));
            k_axpy<<<G, kBlock, 0, s>>>(n, b, tau, t0);
            HNS_TRY(check("axpy"));
        }
        if (f_dev && c < 2) {  // Coriolis: +tau M (f u_2) for c = 1, -tau M (f u_1) for c = 2
            k_hadamard<<<G, kBlock, 0, s>>>(n, t1, f_dev, u_dev + (c == 0 ? 1 : 0) * n);
            HNS_TRY(check("hadamard"));
            HNS_TRY(launch_spmv_plain(op->M, false, t1, t0, nullptr, -1, s));
            k_axpy<<<G, kBlock, 0, s>>>(n, b, c == 0 ? tau : -tau, t0);
            HNS_TRY(check("axpy"));
        }
        if (adv_dev) {                                                     // - tau N_c(u)
            k_axpy<<<G, kBlock, 0, s>>>(n, b, -tau, adv_dev + c * n);
            HNS_TRY(check("axpy"));
        }
        if (p_dev) {                                                       // + tau B_c^T p
            HNS_TRY(apply_div(op, c, true, p_dev, t0, s));
            k_axpy<<<G, kBlock, 0, s>>>(n, b, tau, t0);
            HNS_TRY(check("axpy"));
        }
        if (op->bc) {
            k_mask<<<G, kBlock, 0, s>>>(n, b, op->bc, c);
            HNS_TRY(check("mask"));
        }
    }
    HNS_TRY_HIP(hipStreamSynchronize(s));
    return HNS_OK;
}

hns_status hns_step_pressure_rhs_tau(hns_operator *op, double tau, const double *ut_dev,
                                     double *b_dev, void *stream)
{
    HNS_TRY(need_aux(op));
    if (!ut_dev || !b_dev || !(tau != 0.0) || !std::isfinite(tau)) {
        set_error("hns_step_pressure_rhs_tau: null vector or zero time step");
        return HNS_ERR_INVALID;
    }
    return pressure_rhs(op, -1.0 / tau, ut_dev, b_dev, (hipStream_t)stream);
}

static hns_status pressure_rhs(hns_operator *op, double scale, const double *ut_dev,
                               double *b_dev, hipStream_t s)
{
    const int64_t n = op->n;
    const int G = stream_grid(n);
    if (op->Bdia && !overlaps(ut_dev, 3 * n, b_dev, n)) {
        const FormArgs f = form_args(op);
        k_pressure_rhs<<<form_grid(n), kBlock, 0, s>>>(f, scale, ut_dev, b_dev);
        HNS_TRY(check("pressure rhs"));
        HNS_TRY_HIP(hipStreamSynchronize(s));
        return HNS_OK;
    }
    std::lock_guard<std::mutex> scratch(op->step_mutex);
    double *t0 = op->step_tmp;
    for (int c = 0; c < 3; ++c) {
        HNS_TRY(apply_div(op, c, false, ut_dev + c * n, t0, s));
        if (c == 0)
            k_scale<<<G, kBlock, 0, s>>>(n, b_dev, scale, t0);
        else
            k_axpy<<<G, kBlock, 0, s>>>(n, b_dev, scale, t0);
        HNS_TRY(check("pressure rhs"));
    }
    HNS_TRY_HIP(hipStreamSynchronize(s));
    return HNS_OK;
}

hns_status hns_step_correct_rhs(hns_operator *op, double tau, const double *ut_dev,
                                const double *q_dev, double *p_dev, double *rhs_dev,
                                void *stream)
{
    HNS_TRY(need_aux(op));
    if (!ut_dev || !q_dev || !rhs_dev || !std::isfinite(tau)) {
        set_error("hns_step_correct_rhs: null vector or non-finite time step");
        return HNS_ERR_INVALID;
    }
    hipStream_t s = (hipStream_t)stream;
    if (op->Bdia && !overlaps(rhs_dev, 3 * op->n, ut_dev, 3 * op->n) &&
        !overlaps(rhs_dev, 3 * op->n, q_dev, op->n) &&
        p_alone(op->n, p_dev, q_dev, ut_dev, rhs_dev)) {
        const FormArgs f = form_args(op);
        k_correct_rhs<<<form_grid(f.n), kBlock, 0, s>>>(f, tau, ut_dev, q_dev, p_dev, rhs_dev);
        HNS_TRY(check("correction right-hand side"));
        HNS_TRY_HIP(hipStreamSynchronize(s));
        return HNS_OK;
    }
    const int64_t n = op->n;
    const int G = stream_grid(n);
    std::lock_guard<std::mutex> scratch(op->step_mutex);
    double *t0 = op->step_tmp, *t1 = op->step_tmp + n;
    if (p_dev) {
        k_axpy<<<G, kBlock, 0, s>>>(n, p_dev, 1.0, q_dev);
        HNS_TRY(check("pressure update"));
    }
    for (int c = 0; c < 3; ++c) {
        double *r = rhs_dev + c * n;
        HNS_TRY(launch_spmv_plain(op->M, false, ut_dev + c * n, t0, nullptr, -1, s));
        HNS_TRY(apply_div(op, c, false, q_dev, t1, s));
        k_axpy<<<G, kBlock, 0, s>>>(n, t0, -tau, t1);
        HNS_TRY(check("axpy"));
        k_copy_masked<<<G, kBlock, 0, s>>>(n, r, t0, op->bc, op->bc ? c : -1);
        HNS_TRY(check("mask"));
    }
    HNS_TRY_HIP(hipStreamSynchronize(s));
    return HNS_OK;
}

}  // extern "C"
