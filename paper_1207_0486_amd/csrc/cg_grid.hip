// A chunk of Jacobi-scaled CG iterations in one launch: one workgroup per CU,
// the rows split into tiles whose vectors stay on chip for the whole chunk.
//
// A launch per phase (spmv, update, direction update) streams every vector
// through memory three times per iteration and pays two or three launch
// boundaries; up to about 800 rows per CU those boundaries are the whole cost
// and at 1.4M rows the vectors are 60 % of the bytes.  Here a workgroup keeps
// its rows' r and x and as many matrix values as fit in registers, its p (and
// the p of the rows its products reach) in LDS, and the workgroups meet twice
// per iteration, once per dot product.  What crosses between workgroups is
// the partial sums and q on the tiles' edges.
//
// Tiles.  The offsets of the layered meshes form two groups: |o| <= H within
// a plane of P rows, and P + d, |d| <= H, to the next plane.  Row i is (plane
// i / P, place i % P), and a tile is A planes by S places: its products reach
// one plane above and below and H places to either side.  (A strip of whole
// planes would reach 2 P rows: 10.8K at 256x256x20, where a tile of 5.4K rows
// reaches 1.5K.)  Row numbers stay linear, so a place outside 0..P-1 is
// simply the row i = plane P + place; a matrix whose offsets do not fall into
// such groups is one plane of n rows.
//
// Meeting.  Every workgroup posts its partial sums as 64-bit words (32 bits
// of a double, 32 bits of the meeting's number) with device-scope stores and
// polls the others' words until their numbers match: data and arrival are one
// word, so no counter, no fence and no reset.  Two sets of slots alternate; a
// workgroup can post meeting k + 2 only after every other has posted k + 1,
// that is, has read k.  Up to 64 workgroups one wavefront polls a slot per lane, up
// to 128 a wavefront every 16 slots, beyond that the sums go through groups of 16.
// Measured per meeting of one / two sums on MI355X: 1.7 / 1.8 us among 64
// workgroups, 1.9 / 2.0 among 128, 2.2 / 2.4 among 256 through the groups (3.2
// with every workgroup polling 256 slots, 7.3 with the slots side by side
// instead of 256 bytes apart).  All sums are in a
// fixed order, so every workgroup holds bit-identical scalars and takes the
// same decisions.
//
// q on the tiles' edges is stored with device scope during the product and
// complete before the partial sum is posted; a workgroup reads its
// neighbours' q between the meetings (the latency hides behind the second),
// and updates their r and p itself by the expressions their owners use, bit
// for bit.  Two buffers alternate (q and p, whose memory the chunk does not
// use otherwise).
//
// Progress.  The workgroups wait for each other, so all of a launch must become
// resident.  One takes a CU at most (512 threads, up to 256 registers), and a launch of G is
// dealt round-robin to the 8 XCDs and the 4 shader engines of each: at most
// ceil(G / 32) to an engine.  The caller admits launches while the sum of these
// counts is at most the CUs of an engine (GridTurn in solve.hip), so each finds its
// CUs as soon as kernels that do not wait have left them.  (hipLaunchCooperativeKernel
// would run one such launch at a time, whatever its size, and block the calling
// thread until it ends: eight threads solving 41,664 rows each got 192 solves per
// second that way, 370 with launches per phase.)  A poll is bounded all the same:
// on running out, the workgroup raises Scalars::lost and leaves, the others run out
// in turn, and the caller repeats the segment with a launch per phase: r, p and x are
// void then, and x is the segment's correction (some forms update it in memory in
// every iteration), never the caller's x, so nothing is lost but time.
#include <algorithm>
#include <cmath>

#include "device_util.h"
#include "kernels.h"

namespace hns {
namespace {

constexpr int kGT = kGridBlock;         // threads of a workgroup
constexpr int kGW = kGT / 64;           // its wavefronts
constexpr int kSlotWords = 32;          // 64-bit words between two slots
constexpr int kGroup = 16;              // workgroups of a summing group
constexpr int kFlat = kGW * kGroup;     // up to this many workgroups: no groups
constexpr int kHaloMax = 4;             // edge rows per thread

template <typename TX>
struct GridArgs {
    int64_t n;
    int32_t P, planes, A, S, nS, nch, H, pitch, hcap;
    uint32_t inv_nch;         // 2^20 / nch, rounded up: u / nch for u < 1024
    int32_t off[kGridDiag];   // row offsets of the upper diagonals
    int32_t dl[kGridDiag];    // the same in LDS places
    const TX *dia;
    TX *x, *r, *p, *q;
    const float *w;
    const uint8_t *bc;
    int bit;
    Scalars *sc;
    uint64_t *slots;
    int parity, count, wlds;
    int polls;   // polls before a meeting is given up
};

__device__ __forceinline__ void post64(uint64_t *p, uint64_t v)
{
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

__device__ __forceinline__ uint64_t peek64(const uint64_t *p)
{
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Words of NV doubles into a slot: one store of 2 NV lanes, so the words go out
// as one write (a store per word took 0.8 us more per meeting of two sums).
// v is the same in every lane.
template <int NV>
__device__ __forceinline__ void post(uint64_t *slot, uint32_t tag, const double (&v)[NV], int lane)
{
    const double first = v[0], second = v[NV - 1];
    const double d = lane < 2 ? first : second;
    const uint32_t w = (lane & 1) ? __double2hiint(d) : __double2loint(d);
    if (lane < 2 * NV) post64(slot + lane, (uint64_t)tag << 32 | w);
}

// The sums over `count` <= kGroup slots, in every lane, once all their words
// carry `tag`: a word per lane, so a poll is one load.  False after `polls`.
template <int NV>
__device__ __forceinline__ bool collect(const uint64_t *slots, int count, uint32_t tag, int polls,
                                        double (&v)[NV], int lane)
{
    static_assert(2 * NV * kGroup <= 64, "a lane per word");
    const int slot = lane / (2 * NV), word = lane % (2 * NV);
    const uint64_t *p = slots + (size_t)slot * kSlotWords + word;
    uint64_t u = 0;
    bool ok = slot >= count;
    for (int spin = 0; spin < polls; ++spin) {
        if (!ok) {
            u = peek64(p);
            ok = (uint32_t)(u >> 32) == tag;
        }
        if (__all(ok)) break;
    }
    if (!__all(ok)) return false;
    // even lanes: this lane's word is the low half, the next lane's the high
    const int w = (int)(uint32_t)u;
    const int next = __builtin_amdgcn_update_dpp(0, w, 0xB1, 0xf, 0xf, true);   // lane ^ 1
    const double d = __hiloint2double(next, w);
#pragma unroll
    for (int k = 0; k < NV; ++k) v[k] = wave_sum(slot < count && word == 2 * k ? d : 0.0);
    return true;
}

// The same over up to 64 slots, a slot per lane.
template <int NV>
__device__ __forceinline__ bool collect_few(const uint64_t *slots, int count, uint32_t tag,
                                            int polls, double (&v)[NV], int lane)
{
    const uint64_t *p = slots + (size_t)lane * kSlotWords;
    uint64_t u[2 * NV];
    bool ok = lane >= count;
#pragma unroll
    for (int k = 0; k < 2 * NV; ++k) u[k] = 0;
    for (int spin = 0; spin < polls; ++spin) {
        if (!ok) {
#pragma unroll
            for (int k = 0; k < 2 * NV; ++k) u[k] = peek64(p + k);
            ok = true;
#pragma unroll
            for (int k = 0; k < 2 * NV; ++k) ok = ok && (uint32_t)(u[k] >> 32) == tag;
        }
        if (__all(ok)) break;
    }
    if (!__all(ok)) return false;
#pragma unroll
    for (int k = 0; k < NV; ++k)
        v[k] = wave_sum(lane < count ? __hiloint2double((int)(uint32_t)u[2 * k + 1],
                                                        (int)(uint32_t)u[2 * k])
                                     : 0.0);
    return true;
}

__device__ __forceinline__ int fresh_scalar(int v)
{
    asm volatile("" : "+s"(v));
    return v;
}

// base[i] with a 32-bit byte offset (an array shorter than 4 GB)
template <typename T>
__device__ __forceinline__ T at32(const T *base, uint32_t i)
{
    return *reinterpret_cast<const T *>(reinterpret_cast<const char *>(base) +
                                        i * (uint32_t)sizeof(T));
}

struct GridShared {
    double red[2][kGW][2];
    double tot[2][kGW][2];
    int bad;
};

// One meeting: v becomes the sum over all threads of all workgroups.  STORED:
// the device-scope stores made before it are complete when its sums appear.
// meanwhile() runs once in every thread after this workgroup has posted, last
// in the wavefronts that poll.
template <int NV, bool STORED, typename F>
__device__ __forceinline__ bool meet(uint64_t *slots, int G, int lb, uint32_t tag, int polls,
                                     double (&v)[NV], GridShared &sh, F &&meanwhile)
{
    const int lane = fresh(threadIdx.x & 63);
    const int wid = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int par = tag & 1;
#pragma unroll
    for (int k = 0; k < NV; ++k) v[k] = wave_sum(v[k]);
    if (lane == 0) {
#pragma unroll
        for (int k = 0; k < NV; ++k) sh.red[par][wid][k] = v[k];
    }
    // this wavefront's device-scope stores have reached memory
    if constexpr (STORED) asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
    uint64_t *set = slots + (size_t)par * kGridSlots * kSlotWords;
    uint64_t *groups = set + (size_t)kGridMaxWg * kSlotWords;
    const bool few = G <= 64;
    const int ng = few ? 1 : (G + kGroup - 1) / kGroup;
    const bool flat = ng <= kGW;
    if (wid == 0) {
        double own[NV];
#pragma unroll
        for (int k = 0; k < NV; ++k) {
            own[k] = 0.0;
            for (int w = 0; w < kGW; ++w) own[k] += sh.red[par][w][k];
        }
        post<NV>(set + (size_t)lb * kSlotWords, tag, own, lane);
    }
    // a group's leader sums the group; the first wavefronts poll what the
    // total is made of
    const bool leads = !flat && wid == 1 && lb % kGroup == 0;
    const bool polls_total = flat ? wid < ng : wid == 0;
    if (!leads && !polls_total) meanwhile();
    if (leads || polls_total) {
        const int at = leads ? lb : flat ? wid * kGroup : kGridMaxWg;
        const int count = min(kGroup, (at == kGridMaxWg ? ng : G - at));
        double t[NV];
        const bool ok =
            few ? collect_few<NV>(set, G, tag, polls, t, lane)
                : collect<NV>(set + (size_t)at * kSlotWords, count, tag, polls, t, lane);
        if (leads) {
            if (ok) post<NV>(groups + (size_t)(lb / kGroup) * kSlotWords, tag, t, lane);
        } else if (lane == 0) {
#pragma unroll
            for (int k = 0; k < NV; ++k) sh.tot[par][wid][k] = ok ? t[k] : 0.0;
        }
        if (!ok && lane == 0) sh.bad = 1;
        meanwhile();
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < NV; ++k) {
        v[k] = sh.tot[par][0][k];
        if (flat)
            for (int w = 1; w < ng; ++w) v[k] += sh.tot[par][w][k];
    }
    return sh.bad == 0;
}

// Workgroups are dealt to the 8 XCDs round-robin: number them so that each XCD
// holds consecutive ones (the groups' words then stay near)
__device__ __forceinline__ int grid_block(int b, int G)
{
    const int x = b & 7;
    return x * (G >> 3) + min(x, G & 7) + (b >> 3);
}

// RPT: groups of 64 consecutive places (one per wavefront) of a tile, per
// wavefront, at most.  NU, NL: upper and lower diagonals kept in registers
// and ND further lower ones in LDS (the others are read from memory in every
// iteration, a row ahead); XREG: x in registers.
template <typename TX, int M, int RPT, int NU, int NL, int ND, bool XREG, bool AHEAD>
__global__ __launch_bounds__(kGT) __attribute__((amdgpu_waves_per_eu(2, 2)))
void k_cg_grid(GridArgs<TX> g)
{
    extern __shared__ double grid_lds[];
    __shared__ GridShared sh;
    if (g.sc->stop) return;   // written by earlier launches, or by this one's end only
    const int lane = threadIdx.x & 63;
    const int wid = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int G = gridDim.x;
    const int lb = grid_block(blockIdx.x, G);
    const int a0 = (lb / g.nS) * g.A, s0 = (lb % g.nS) * g.S;
    const int A = min(g.A, g.planes - a0), S = min(g.S, g.P - s0);
    const int H = g.H, pitch = g.pitch;
    const int n = (int)g.n;
    const int span = S + 2 * H;                 // places held of a plane
    const int hcount = 2 * span + 2 * H * A;    // edge rows held
    TX *sp = reinterpret_cast<TX *>(grid_lds);
    TX *hr = sp + (size_t)(g.A + 2) * pitch;
    int32_t *hg = reinterpret_cast<int32_t *>(hr + g.hcap);
    int32_t *hl = hg + g.hcap;
    TX *sd = reinterpret_cast<TX *>(hl + g.hcap);
    float *sw = reinterpret_cast<float *>(sd + (size_t)ND * RPT * kGT);

    for (int i = threadIdx.x; i < (g.A + 2) * pitch; i += kGT) sp[i] = (TX)0;
    if (threadIdx.x == 0) sh.bad = 0;
    __syncthreads();
    // the tile's own rows: unit u = wavefront + 8 j is 64 places of one plane,
    // at LDS place lds and row (of the first lane; recomputed in scalar
    // registers where they are used, since the table does not fit beside the
    // rest)
    struct Unit {
        int lds, row, al, c;
        bool in;
    };
    auto unit = [&](int w, int j) {
        Unit q;
        const int u = w + kGW * j;
        q.in = u < A * g.nch;
        const int al = (int)(((uint32_t)u * g.inv_nch) >> 20);
        q.al = q.in ? al : 0;
        q.c = q.in ? u - al * g.nch : 0;
        q.lds = (q.al + 1) * pitch + H + q.c * 64;
        q.row = (a0 + q.al) * g.P + s0 + q.c * 64;
        return q;
    };
    uint32_t live = 0, fixed = 0, edge = 0;   // per row: exists, Dirichlet, read by others
    TX rv[RPT], xv[XREG ? RPT : 1], up[RPT][NU > 0 ? NU : 1], lo[RPT][NL > 0 ? NL : 1];
#pragma unroll
    for (int j = 0; j < RPT; ++j) {
        const Unit q = unit(fresh_scalar(wid), j);
        const int al = q.al, sl = q.c * 64 + lane;
        const int gi = q.row + lane, li = q.lds + lane;
        const bool ex = q.in && sl < S && gi < n;
        if (ex) live |= 1u << j;
        if (!ex || is_dirichlet(g.bc, g.bit, gi)) fixed |= 1u << j;
        if (ex && (al == 0 || al == A - 1 || sl < H || sl >= S - H)) edge |= 1u << j;
        rv[j] = ex ? g.r[gi] : (TX)0;
        if constexpr (XREG) xv[j] = ex ? g.x[gi] : (TX)0;
        if (ex) sp[li] = g.p[gi];
        if (g.wlds) sw[j * kGT + threadIdx.x] = ex ? g.w[gi] : 0.0f;
#pragma unroll
        for (int k = 0; k < NU; ++k) up[j][k] = ex ? at32(g.dia + (int64_t)k * n, gi) : (TX)0;
#pragma unroll
        for (int k = 0; k < NL; ++k)
            lo[j][k] = ex && gi >= g.off[k] ? at32(g.dia + (int64_t)k * n, gi - g.off[k]) : (TX)0;
#pragma unroll
        for (int k = 0; k < ND; ++k)
            sd[(k * RPT + j) * kGT + threadIdx.x] =
                ex && gi >= g.off[NL + k] ? at32(g.dia + (int64_t)(NL + k) * n, gi - g.off[NL + k])
                                          : (TX)0;
        __builtin_amdgcn_sched_barrier(0);
    }
    // the edge rows: the planes below and above, and H places to either side
    for (int h = threadIdx.x; h < hcount; h += kGT) {
        int ap, s;
        if (h < 2 * span) {
            ap = h < span ? 0 : A + 1;
            s = h < span ? h : h - span;
        } else {
            const int e = h - 2 * span;
            ap = 1 + e / (2 * H);
            s = e % (2 * H);
            s = s < H ? s : s + S;
        }
        const int64_t gi = (int64_t)(a0 + ap - 1) * g.P + s0 - H + s;
        const int li = ap * pitch + s;
        const bool ex = gi >= 0 && gi < n;
        hg[h] = ex ? (int32_t)gi : -1;
        hl[h] = li;
        hr[h] = ex ? g.r[gi] : (TX)0;
        if (ex) sp[li] = g.p[gi];
    }
    const double thr = g.sc->tol2 * g.sc->bb;
    double rho = g.sc->rho[g.parity], rho_prev = rho, rr = 0.0, alpha_d = 0.0, beta_d = 0.0,
           gamma = 0.0;
    int done = 0, stop = 0;
    bool lost = false;
    __syncthreads();

    for (int it = 0; it < g.count; ++it) {
        TX *pub = (it & 1) ? g.p : g.q;
        TX qv[RPT];
        double acc = 0.0;
        int ln = fresh(lane), ws = fresh_scalar(wid);
        const int tn = fresh(threadIdx.x);
        uint32_t fx = fresh(fixed), eg = fresh(edge);
        constexpr int FU = M - NU, FL = M - NL - ND;   // diagonals read from memory
        TX us[2][FU > 0 ? FU : 1], ls[2][FL > 0 ? FL : 1];
        auto fetch = [&](int j, int to) {
            const int gc = min(unit(ws, j).row + ln, n - 1);   // past the end: loaded, then dropped
#pragma unroll
            for (int k = 0; k < FU; ++k) us[to][k] = at32(g.dia + (int64_t)(NU + k) * n, gc);
#pragma unroll
            for (int k = 0; k < FL; ++k)
                ls[to][k] = at32(g.dia + (int64_t)(NL + ND + k) * n, max(gc - g.off[NL + ND + k], 0));
        };
        // p of a row and of the 2 M rows it couples to
        TX pc[AHEAD ? 2 : 1], pu[AHEAD ? 2 : 1][M], pl[AHEAD ? 2 : 1][M];
        auto gather = [&](int j, int to) {
            const TX *pj = sp + unit(ws, j).lds + ln;
            pc[to] = pj[0];
#pragma unroll
            for (int k = 0; k < M; ++k) {
                pu[to][k] = pj[g.dl[k]];
                pl[to][k] = pj[-g.dl[k]];
            }
        };
        fetch(0, 0);
        if constexpr (AHEAD) gather(0, 0);
#pragma unroll
        for (int j = 0; j < RPT; ++j) {
            if (j + 1 < RPT) fetch(j + 1, (j + 1) & 1);
            if (AHEAD) {
                if (j + 1 < RPT) gather(j + 1, (j + 1) & 1);
            } else {
                gather(j, 0);
            }
            __builtin_amdgcn_sched_barrier(0);
            const int at = AHEAD ? j & 1 : 0;
            const int gi = unit(ws, j).row + ln;
            const TX pi = pc[at];
            TX sum = pi;
#pragma unroll
            for (int k = 0; k < M; ++k) {
                const TX uv = k < NU                 ? up[j][k < NU ? k : 0]
                              : gi + g.off[k] < n ? us[j & 1][k >= NU ? k - NU : 0]
                                                  : (TX)0;
                const TX lv = k < NL           ? lo[j][k < NL ? k : 0]
                              : k < NL + ND    ? sd[((k - NL) * RPT + j) * kGT + tn]
                              : gi >= g.off[k] ? ls[j & 1][k >= NL + ND ? k - NL - ND : 0]
                                               : (TX)0;
                sum += uv * pu[at][k];
                sum += lv * pl[at][k];
            }
            if ((fx >> j) & 1u) sum = (TX)0;
            qv[j] = sum;
            acc += (double)pi * (double)sum;
            if ((eg >> j) & 1u)
                __hip_atomic_store(pub + gi, sum, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            __builtin_amdgcn_sched_barrier(0);
        }
        double v1[1] = {acc};
        if (!meet<1, true>(g.slots, G, lb, 2 * it + 1, g.polls, v1, sh, [] {})) {
            lost = true;
            break;
        }
        gamma = v1[0];
        if (!(gamma > 0.0) || !isfinite(gamma)) {
            stop = 2;
            break;
        }
        alpha_d = rho / gamma;
        const TX alpha = (TX)alpha_d;
        const bool last = it + 1 == g.count;
        TX hq[kHaloMax];
        int tid = fresh(threadIdx.x);
#pragma unroll
        for (int m = 0; m < kHaloMax; ++m) {
            const int h = tid + kGT * m;
            hq[m] = (TX)0;
            if (!last && h < hcount) {
                const int gi = hg[h];
                if (gi >= 0)
                    hq[m] = __hip_atomic_load(pub + gi, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            }
        }
        double v2[2] = {0.0, 0.0};
        ln = fresh(lane);
        ws = fresh_scalar(wid);
        uint32_t lv = fresh(live);
#pragma unroll
        for (int j = 0; j < RPT; ++j) {
            rv[j] = fma_t(-alpha, qv[j], rv[j]);
            const double ri = (double)rv[j];
            const float wi = g.wlds ? sw[j * kGT + tid]
                                    : ((lv >> j) & 1u) ? at32(g.w, unit(ws, j).row + ln) : 0.0f;
            v2[0] += ri * ri;
            v2[1] += (double)wi * ri * ri;
        }
        const bool met = meet<2, false>(g.slots, G, lb, 2 * it + 2, g.polls, v2, sh, [&] {
            const int t = fresh(threadIdx.x), l2 = fresh(lane), w2 = fresh_scalar(wid);
            const uint32_t v = fresh(live);
#pragma unroll
            for (int m = 0; m < kHaloMax; ++m) {
                const int h = t + kGT * m;
                if (h < hcount) hr[h] = fma_t(-alpha, hq[m], hr[h]);
            }
            if constexpr (XREG) {
#pragma unroll
                for (int j = 0; j < RPT; ++j)
                    xv[j] = fma_t(alpha, sp[unit(w2, j).lds + l2], xv[j]);
            } else {
                constexpr int B = 4;   // loads in flight
#pragma unroll
                for (int j0 = 0; j0 < RPT; j0 += B) {
                    TX xo[B];
#pragma unroll
                    for (int j = j0; j < j0 + B && j < RPT; ++j)
                        if ((v >> j) & 1u) xo[j - j0] = g.x[unit(w2, j).row + l2];
#pragma unroll
                    for (int j = j0; j < j0 + B && j < RPT; ++j)
                        if ((v >> j) & 1u)
                            g.x[unit(w2, j).row + l2] =
                                fma_t(alpha, sp[unit(w2, j).lds + l2], xo[j - j0]);
                    __builtin_amdgcn_sched_barrier(0);
                }
            }
        });
        if (!met) {
            lost = true;
            break;
        }
        rr = v2[1];
        beta_d = v2[0] / rho;
        rho_prev = rho;
        rho = v2[0];
        ++done;
        if (!isfinite(rho) || !isfinite(rr)) {
            stop = 2;
            break;
        }
        if (rr <= thr) {
            stop = 1;
            break;
        }
        const TX beta = (TX)beta_d;
        ln = fresh(lane);
        lv = fresh(live);
        ws = fresh_scalar(wid);
        tid = fresh(threadIdx.x);
#pragma unroll
        for (int j = 0; j < RPT; ++j)
            if ((lv >> j) & 1u) {
                TX *pj = sp + unit(ws, j).lds + ln;
                *pj = fma_t(beta, *pj, rv[j]);
            }
#pragma unroll
        for (int m = 0; m < kHaloMax; ++m) {
            const int h = tid + kGT * m;
            if (h < hcount) sp[hl[h]] = fma_t(beta, sp[hl[h]], hr[h]);
        }
        __syncthreads();
    }

    if (lost) {
        if (threadIdx.x == 0) g.sc->lost = 1;
        return;
    }
#pragma unroll
    for (int j = 0; j < RPT; ++j)
        if ((live >> j) & 1u) {
            const Unit q = unit(fresh_scalar(wid), j);
            const int gi = q.row + lane;
            g.r[gi] = rv[j];
            g.p[gi] = sp[q.lds + lane];
            if constexpr (XREG) g.x[gi] = xv[j];
        }
    if (lb == 0 && threadIdx.x == 0) {
        Scalars *sc = g.sc;
        if (done > 0) {
            sc->rho[(g.parity + done - 1) & 1] = rho_prev;
            sc->rho[(g.parity + done) & 1] = rho;
            sc->rr = rr;
            sc->beta = beta_d;
            sc->iter += done;
        }
        sc->alpha = alpha_d;
        sc->gamma = gamma;
        if (stop) sc->stop = stop;
    }
}

__global__ __launch_bounds__(kBlock) void k_clear_slots(uint64_t *slots, int words)
{
    for (int i = blockIdx.x * kBlock + threadIdx.x; i < words; i += gridDim.x * kBlock)
        slots[i] = 0;
}

template <typename TX>
using GridKernel = void (*)(GridArgs<TX>);

// The instances, by rows per thread (a multiple of 512 rows per workgroup
// each).  As many diagonals stay in registers as 256 of them per lane hold.
template <typename TX>
struct Instance {
    int rpt;
    int in_lds;     // lower diagonals in LDS
    int streamed;   // diagonals read from memory in every iteration
    bool xreg;      // x in registers
    GridKernel<TX> k;
};

template <typename TX, int RPT, int NU, int NL, int ND, bool XREG, bool AHEAD>
Instance<TX> instance()
{
    return {RPT, ND, 14 - NU - NL - ND, XREG, k_cg_grid<TX, kGridDiag, RPT, NU, NL, ND, XREG, AHEAD>};
}

const Instance<double> *instances(int *count, double)
{
    static const Instance<double> t[] = {
        instance<double, 1, 7, 7, 0, true, false>(), instance<double, 2, 7, 7, 0, true, true>(),
        instance<double, 4, 7, 7, 0, true, true>(),  instance<double, 6, 7, 5, 2, false, false>(),
        instance<double, 8, 7, 2, 2, false, false>(),
        instance<double, 12, 4, 0, 1, false, false>(),
    };
    *count = sizeof(t) / sizeof(t[0]);
    return t;
}

const Instance<float> *instances(int *count, float)
{
    static const Instance<float> t[] = {
        instance<float, 1, 7, 7, 0, true, false>(), instance<float, 2, 7, 7, 0, true, true>(),
        instance<float, 4, 7, 7, 0, true, true>(),  instance<float, 8, 7, 7, 0, true, true>(),
        instance<float, 12, 7, 5, 2, false, true>(),
    };
    *count = sizeof(t) / sizeof(t[0]);
    return t;
}

constexpr size_t kLdsMax = 160 * 1024 - sizeof(GridShared) - 256;

size_t lds_bytes(const GridPlan &p, size_t vb, int rpt, int in_lds, bool wlds)
{
    return (size_t)(p.A + 2) * p.pitch * vb + (size_t)p.hcap * (vb + 8) +
           (size_t)in_lds * rpt * kGT * vb +
           (wlds ? (size_t)rpt * kGT * sizeof(float) : 0);
}

// Time of one iteration of a plan in us, fitted to phases timed on MI355X: two
// meetings; product, r and p updates per 512 rows of a workgroup (LDS latency
// more than its rate: FP32 and FP64 alike); what is read from memory, at the
// 8.7 TB/s such reads reached (they stay in the caches between iterations: 129 MB
// at 256x256x20, 108 MB at 250x200x22).  Estimated / measured in FP64, us: 7.8 / 7.6
// at 160x140x20, 10.0 / 9.6 at 200x180x20, 12.9 / 12.3 at 240x189x17, 22.6 / 22.7 at
// 250x200x22, 25.7 / 25.5 at 256x256x20.
double plan_cost(int G, int rpt, int streamed, bool xreg, int halo, size_t vb)
{
    const double meet = G <= 64 ? 3.6 : G <= kFlat ? 4.6 : 5.4;
    const double mem = streamed * vb + (xreg ? 0.0 : 2.0 * vb);
    return meet + 0.6 + 0.37 * rpt + G * kGT * (double)rpt * mem / 8.7e6 + 0.15 * halo / kGT;
}

template <typename TX>
bool plan_for(const DevMatrix &S, int cus, GridPlan &best)
{
    best = GridPlan{};
    if (!S.unit || S.fmt != HNS_FMT_SDIA || S.ndiag != 7 || S.n >= (1 << 30)) return false;
    int count = 0;
    const Instance<TX> *inst = instances(&count, TX());
    const int64_t n = S.n;
    const int m = S.ndiag;
    const int wgs = std::min(cus, kGridMaxWg);
    best.cost = 1e30;
    for (int split = 1; split <= m; ++split) {   // diagonals split.. reach the next plane
        int64_t P = n, H = S.off[m - 1];
        if (split < m) {
            P = S.off[split];
            H = std::max<int64_t>(S.off[split - 1], S.off[m - 1] - P);
            if (P < 2 * H) continue;   // a plane must be wider than what is reached within it
        }
        const int64_t planes = (n + P - 1) / P;
        for (int64_t nch = 1; nch <= (P + 63) / 64; ++nch) {
            const int64_t Sw = nch * 64, nS = (P + Sw - 1) / Sw, pitch = Sw + 2 * H;
            if (nS > wgs || pitch * 3 * sizeof(TX) > kLdsMax) continue;
            for (int64_t nA = std::min<int64_t>(planes, wgs / nS); nA >= 1; --nA) {
                const int64_t A = (planes + nA - 1) / nA;
                const int64_t units = A * nch, rows = (units + kGW - 1) / kGW;
                if (rows > inst[count - 1].rpt) break;   // larger tiles only from here on
                const int64_t halo = 2 * pitch + 2 * H * A;
                if (halo > (int64_t)kHaloMax * kGT) continue;
                int i = 0;
                while (inst[i].rpt < rows) ++i;
                GridPlan p;
                p.A = (int)A;
                p.pitch = (int)pitch;
                p.hcap = (int)((halo + 1) & ~int64_t(1));
                p.wlds = lds_bytes(p, sizeof(TX), inst[i].rpt, inst[i].in_lds, true) <= kLdsMax;
                p.lds = lds_bytes(p, sizeof(TX), inst[i].rpt, inst[i].in_lds, p.wlds);
                if (p.lds > kLdsMax) continue;
                p.G = (int)(((planes + A - 1) / A) * nS);
                p.cost = plan_cost(p.G, (int)rows, inst[i].streamed, inst[i].xreg, (int)halo, sizeof(TX));
                if (p.cost >= best.cost) continue;
                p.P = (int)P;
                p.planes = (int)planes;
                p.S = (int)Sw;
                p.nS = (int)nS;
                p.nch = (int)nch;
                p.H = (int)H;
                p.instance = i;
                p.rpt = inst[i].rpt;
                p.streamed = inst[i].streamed + (inst[i].xreg ? 0 : 2);
                for (int k = 0; k < m; ++k)
                    p.dl[k] = k < split ? S.off[k] : (int)(pitch + S.off[k] - P);
                best = p;
            }
        }
    }
    return best.G > 0;
}

template <typename TX>
hns_status launch_t(const IterArgs &a, const GridPlan &p, int parity, int count, int polls,
                    bool *refused, hipStream_t s)
{
    const DevMatrix &S = *a.A;
    int ni = 0;
    const Instance<TX> *inst = instances(&ni, TX());
    GridArgs<TX> g{};
    g.n = a.n;
    g.P = p.P;
    g.planes = p.planes;
    g.A = p.A;
    g.S = p.S;
    g.nS = p.nS;
    g.nch = p.nch;
    g.inv_nch = ((1u << 20) + p.nch - 1) / p.nch;
    g.H = p.H;
    g.pitch = p.pitch;
    g.hcap = p.hcap;
    for (int k = 0; k < S.ndiag; ++k) {
        g.off[k] = S.off[k];
        g.dl[k] = p.dl[k];
    }
    if constexpr (sizeof(TX) == 8)
        g.dia = S.dia;
    else
        g.dia = S.dia32;
    g.x = (TX *)a.x;
    g.r = (TX *)a.r;
    g.p = (TX *)a.p;
    g.q = (TX *)a.q;
    g.w = a.wjac;
    g.bc = a.bit < 0 ? nullptr : a.bc;
    g.bit = a.bit < 0 ? 0 : a.bit;
    g.sc = a.sc;
    g.slots = (uint64_t *)a.partials;
    g.parity = parity & 1;
    g.count = count;
    g.wlds = p.wlds;
    g.polls = polls;
    const int words = 2 * kGridSlots * kSlotWords;
    k_clear_slots<<<(words + kBlock - 1) / kBlock, kBlock, 0, s>>>(g.slots, words);
    HNS_TRY_HIP(hipGetLastError());
    void *args[] = {&g};
    *refused = hipLaunchKernel((const void *)inst[p.instance].k, dim3(p.G), dim3(kGT), args, p.lds,
                               s) != hipSuccess;
    if (*refused) (void)hipGetLastError();
    return HNS_OK;
}

// The limit on an instance's dynamic LDS belongs to the process: it is set to the
// most that any tiling takes, so that operators planned one after the other, or at
// the same time, do not lower it below what another launches with.
template <typename TX>
bool ready(GridPlan &p)
{
    int ni = 0, blocks = 0;
    const Instance<TX> *inst = instances(&ni, TX());
    const void *k = (const void *)inst[p.instance].k;
    if (hipFuncSetAttribute(k, hipFuncAttributeMaxDynamicSharedMemorySize, (int)kLdsMax) !=
            hipSuccess ||
        hipOccupancyMaxActiveBlocksPerMultiprocessor(&blocks, k, kGT, p.lds) != hipSuccess) {
        (void)hipGetLastError();
        return false;
    }
    return blocks >= 1;
}

}  // namespace

void grid_plans(DevMatrix &S)
{
    static_assert((size_t)2 * kGridSlots * kSlotWords <= (size_t)kPartTotal,
                  "the slots use the partial-sum buffer");
    static_assert(kGridSlots >= kGridMaxWg + kGridMaxWg / kGroup, "slots of the groups");
    S.grid64 = S.grid32 = GridPlan{};
    int dev = 0, cus = 0;
    if (hipGetDevice(&dev) != hipSuccess ||
        hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess) {
        (void)hipGetLastError();
        return;
    }
    cus = cus / kGridEngines * kGridEngines;   // as many on every shader engine
    if (cus == 0) return;
    if (!plan_for<double>(S, cus, S.grid64) || !ready<double>(S.grid64)) S.grid64 = GridPlan{};
    if (S.dia32 && (!plan_for<float>(S, cus, S.grid32) || !ready<float>(S.grid32)))
        S.grid32 = GridPlan{};
    S.grid64.dev = S.grid32.dev = dev;
    S.grid64.room = S.grid32.room = cus / kGridEngines;
}

hns_status launch_cg_grid(const IterArgs &a, int parity, int count, int polls, bool *refused,
                          hipStream_t s)
{
    *refused = false;
    if (count <= 0) return HNS_OK;
    const GridPlan &p = a.prec == Prec::F32 ? a.A->grid32 : a.A->grid64;
    if (p.G <= 0 || !a.wjac || (a.prec != Prec::F64 && a.prec != Prec::F32)) {
        set_error("launch_cg_grid: unsupported configuration");
        return HNS_ERR_INVALID;
    }
    return a.prec == Prec::F64 ? launch_t<double>(a, p, parity, count, polls, refused, s)
                               : launch_t<float>(a, p, parity, count, polls, refused, s);
}

}  // namespace hns
