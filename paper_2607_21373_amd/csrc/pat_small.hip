// Resident sweeps of small meshes: one launch carries a whole N_T-step sweep.
//
// A step of a mesh of a few thousand nodes is launch- and latency-bound: each step
// kernel takes 3 to 8 us whatever its work.  Here one workgroup owns one right-hand
// side for the whole sweep.  The state lives in LDS (three rotating vectors, and two of
// its increments, which the boundary part reads), every thread keeps in registers the
// padded stiffness rows it owns (RPT rows of 16 weights and 16 LDS offsets), their state,
// records, first B values and overflow columns, and the rest of the boundary, overflow
// and sensor tables sit in LDS.  So a step is 15 LDS reads per row and one barrier, with
// no launch and no traffic but the sensor data.  Right-hand sides are independent, so
// workgroups never wait for each other.  A row's arithmetic is the step kernels'
// (pat_step.h, in their slot order), and so are the bits.
//
// Bound: the barrier waits for the wave with the longest chain, the one with overflow
// rows, and for the LDS reads of the CU that holds the right-hand side (15 gathers per
// row, at several cycles each for the bank conflicts of their addresses; without the
// special rows a step of 729 nodes takes 0.7 us).  The overflow entries in a loop of four
// took two dependent LDS reads a turn (an 11-entry row: 0.5 us of a step); with their
// columns in registers all reads of a group go out together.  Measured per forward /
// transposed step: 729 nodes, one float64 RHS 1.05 / 1.29 us (3.0 / 3.2 as step launches;
// 1.58 / 1.81 with records, B values and overflow columns read from LDS), 16 RHS 1.04 /
// 1.19 (6.9 / 7.5; 1.65 / 1.91); 1,331 nodes, one float32 RHS 1.33 / 1.46 (1.64 / 1.92
// from LDS); 2,028 nodes, 16 float32 RHS 1.64 / 1.75 (7.8 / 7.9; 1.88 / 1.95).
#include <hip/hip_runtime.h>

#include <algorithm>

#include "pat_kernels.h"
#include "pat_step.h"

namespace pat {
namespace {

constexpr size_t kLdsBytes = 163840;

constexpr int kOverRegs = 12;  // overflow entries whose columns a thread of one row keeps in registers

// LDS behind the three state vectors (bytes from the start): two vectors of the state's
// increments, the records of the rows with more than padded slots, the B values by
// boundary row, the overflow entries, and forward the sensor rows, transposed the sensor
// weights by node and the ring of sensor data
struct SmallLds {
    size_t inc, rec, bw, xv, xc, sw, sn, iw, is, ring, total;
};
struct SmallSizes {
    int n, n_obs, n_spec, n_bnd, max_nb, n_x, n_inj;
    __host__ __device__ int nb4() const { return (max_nb + 3) / 4 * 4; }
};
template <typename T>
__host__ __device__ inline SmallLds small_lds(int cap, const SmallSizes &z, bool fwd) {
    auto up = [](size_t b) { return (b + 15) & ~size_t(15); };
    SmallLds l;
    l.inc = up(size_t(3) * cap * sizeof(T));
    l.rec = l.inc + 2 * up(size_t(z.n) * sizeof(T));
    l.bw = l.rec + up(size_t(3) * z.n_spec * sizeof(uint32_t));
    l.xv = l.bw + up(size_t(z.n_bnd) * z.nb4() * sizeof(T));
    l.xc = l.xv + up(size_t(z.n_x + kOverRegs) * sizeof(T));  // rows read kOverRegs values, used or not
    l.sw = l.xc + up(size_t(z.n_x) * sizeof(uint16_t));
    l.sn = l.sw + (fwd ? up(size_t(4) * z.n_obs * sizeof(T)) : 0);
    l.iw = l.sn + (fwd ? up(size_t(4) * z.n_obs * sizeof(uint16_t)) : 0);
    l.is = l.iw + (fwd ? 0 : up(size_t(z.n_inj) * sizeof(T)));
    l.ring = l.is + (fwd ? 0 : up(size_t(z.n_inj) * sizeof(uint16_t)));
    l.total = l.ring + (fwd ? 0 : up(size_t(3) * z.n_obs * sizeof(T)));
    return l;
}

template <typename T>
struct SmallArgs {
    const int32_t *ecol, *xcol, *rspec;
    const int32_t *order, *pos;  // row at each place, place of each row (rows of a kind together)
    const T *eval, *xval, *bslot, *dtm;
    const int4 *spec;
    // forward: sensor rows; transpose: their transpose by node (CSR)
    const int32_t *snode, *injs;
    const T *sw, *injw;
    const T *in;       // forward: p0 [N][RB]
    T *out;            // transpose: the result [N][RB]
    void *y;           // forward: samples out; transpose: data in ([N_T][N_obs][RB])
    double yscale;
    SmallSizes z;
    int n_steps, RB;
    T dt;
};

// Barrier for LDS only: the samples' stores and the data's loads stay in flight.
__device__ __forceinline__ void lds_barrier() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// The tables in LDS that every row may read.
template <typename T>
struct SmallTables {
    const uint32_t *rec;  // B rank | slots with B << 16, first overflow entry | count << 16, first weight | count << 16
    const T *bw, *xv;
    const uint16_t *xc;   // byte offsets of the overflow entries' columns
    int n_spec, nb4;
};

// The rows of one thread: those at places threadIdx.x + u blockDim.x of the order that
// puts rows with overflow entries, boundary rows and sensor rows together, so that few
// waves walk those tables (in the node order nearly every wave of a small mesh has some of
// each).  State vectors are held by place.  SPLIT: the sums of the
// scalar-lane kernels (four partial sums over every fourth slot), for the block widths
// those kernels take; else one sum in slot order.
template <typename T, int RPT, bool SPLIT, bool FWD>
struct SmallRows {
    static constexpr int CAP = RPT * kSmallThreads;
    // what a step would read again from LDS and the registers hold (not with two float64 rows):
    // the row's state and increment, its record, and the first NBR of its B values
    static constexpr bool KEEP = RPT * sizeof(T) <= 8;
    static constexpr int NBR = !KEEP ? 0 : !FWD && SPLIT && RPT * sizeof(T) > 4 ? 4 : 8;
    uint32_t off[RPT][8];  // byte offsets of slots 2j and 2j + 1
    T kv[RPT][16];
    T dm[RPT];
    int sp[RPT];           // 0, or 1 + the row's record
    T own[RPT], inc[RPT];
    uint32_t rb[RPT], rx[RPT], re[RPT];
    T bv[RPT][NBR > 0 ? NBR : 1];
    // byte offsets of overflow entries 2j and 2j + 1 of the first row
    static constexpr int NXR = KEEP ? kOverRegs : 0;
    uint32_t xo[NXR / 2 + 1];

    __device__ __forceinline__ uint32_t slot(int u, int j) const {
        return j & 1 ? off[u][j >> 1] >> 16 : off[u][j >> 1] & 0xFFFFu;
    }

    __device__ __forceinline__ void load(const SmallArgs<T> &a, uint32_t *rec, T *bw) {
#pragma unroll
        for (int u = 0; u < RPT; ++u) {
            const int at = int(threadIdx.x) + u * int(blockDim.x);
            sp[u] = 0;
            rb[u] = rx[u] = re[u] = 0u;
            dm[u] = T(0);
#pragma unroll
            for (int j = 0; j < 16; ++j) kv[u][j] = T(0);
#pragma unroll
            for (int j = 0; j < NBR; ++j) bv[u][j] = T(0);
#pragma unroll
            for (int j = 0; j < NXR / 2 && u == 0; ++j) xo[j] = 0u;
#pragma unroll
            for (int j = 0; j < 8; ++j) off[u][j] = 0u;
            if (at >= a.z.n) continue;
            const int row = a.order[at];
            int32_t c[16];
            T w[16];
#pragma unroll
            for (int p = 0; p < 4; ++p) {
                load_quad(a.ecol + int64_t(row) * 16 + 4 * p, c + 4 * p);
                load_quad(a.eval + int64_t(row) * 16 + 4 * p, w + 4 * p);
            }
#pragma unroll
            for (int j = 0; j < 16; ++j) c[j] = a.pos[c[j]];
#pragma unroll
            for (int j = 0; j < 16; ++j) {  // slot j at quad j % 4, element j / 4
                kv[u][j] = w[4 * (j % 4) + j / 4];
                off[u][j >> 1] |= uint32_t(c[4 * (j % 4) + j / 4] * int(sizeof(T))) << (16 * (j & 1));
            }
#pragma unroll
            for (int j = 0; j < 16; ++j) asm volatile("" : "+v"(kv[u][j]));  // one row's loads at a time
            dm[u] = a.dtm[row];
            if (const int k = a.rspec[row]) {
                const int4 s = a.spec[2 * (k - 1)], v = a.spec[2 * (k - 1) + 1];
                sp[u] = k;
                rb[u] = uint32_t(v.z | s.y << 16);
                rx[u] = uint32_t(s.z | (s.w - s.z) << 16);
                re[u] = uint32_t(v.x | (v.y - v.x) << 16);
                rec[k - 1] = rb[u];
                rec[a.z.n_spec + k - 1] = rx[u];
                rec[2 * a.z.n_spec + k - 1] = re[u];
#pragma unroll
                for (int j = 0; j < NBR; ++j)
                    if (j < s.y) bv[u][j] = a.bslot[s.x + 4 * (j % 4) + j / 4];
                if (u == 0 && s.w > s.z) {
#pragma unroll
                    for (int j = 0; j < NXR; ++j)
                        xo[j >> 1] |= uint32_t(a.pos[a.xcol[min(s.z + j, s.w - 1)]] * int(sizeof(T))) << (16 * (j & 1));
                }
                if (s.y)
                    for (int j = 0; j < a.z.nb4(); ++j)
                        bw[v.z * a.z.nb4() + j] = j < s.y ? a.bslot[s.x + 4 * (j % 4) + j / 4] : T(0);
            }
        }
    }

    // acc = K X and bacc = B D (NEGATE: -B D) of row u, and the row's own X (slot 0)
    template <bool NEGATE>
    __device__ __forceinline__ void sums(int u, const char *X, const char *D, const SmallTables<T> &t, T &acc, T &bacc,
                                         T &cur) {
        // unpacked again in every step: kept apart they would take twice the registers
#pragma unroll
        for (int j = 0; j < 8; ++j) asm volatile("" : "+v"(off[u][j]));
        constexpr int CH = RPT * sizeof(T) > 8 ? 4 : 8;  // reads in flight
        T s[SPLIT ? 4 : 1] = {}, b[SPLIT ? 4 : 1] = {};
#pragma unroll
        for (int j0 = 0; j0 < 16; j0 += CH) {
            T x[CH];
#pragma unroll
            for (int j = 0; j < CH; ++j)
                x[j] = KEEP && j0 + j == 0 ? own[u] : *reinterpret_cast<const T *>(X + slot(u, j0 + j));
            if (j0 == 0) cur = KEEP ? own[u] : x[0];
#pragma unroll
            for (int j = 0; j < CH; ++j) {
                T &o = s[SPLIT ? j % 4 : 0];
                o = mad(kv[u][j0 + j], x[j], o);
            }
            if (CH == 4) __builtin_amdgcn_sched_barrier(0);
        }
        if (sp[u]) {
            const uint32_t rbu = KEEP ? rb[u] : t.rec[sp[u] - 1], rxu = KEEP ? rx[u] : t.rec[t.n_spec + sp[u] - 1];
            const int nb = int(rbu >> 16), nx = int(rxu >> 16), x0 = int(rxu & 0xFFFFu);
            // those past nb have weight 0 in the table and add +0
            const T *w = t.bw + int(rbu & 0xFFFFu) * t.nb4;
            if constexpr (KEEP) {
                if (nb) {
                    T d[NBR];
#pragma unroll
                    for (int j = 0; j < NBR; ++j) d[j] = *reinterpret_cast<const T *>(D + slot(u, j));
#pragma unroll
                    for (int j = 0; j < NBR; ++j) {
                        T &o = b[SPLIT ? j % 4 : 0];
                        o = mad(bv[u][j], j < nb ? (NEGATE ? -d[j] : d[j]) : T(0), o);
                    }
                }
            }
#pragma unroll
            for (int j0 = NBR; j0 < 16; j0 += 4) {  // four slots at a time
                if (j0 >= nb) break;
                T wv[4], d[4];
                load_quad(w + j0, wv);
#pragma unroll
                for (int j = 0; j < 4; ++j) d[j] = *reinterpret_cast<const T *>(D + slot(u, j0 + j));
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    T &o = b[SPLIT ? j : 0];
                    o = mad(wv[j], j0 + j < nb ? (NEGATE ? -d[j] : d[j]) : T(0), o);
                }
            }
            // overflow entries: the columns in registers, XG values at a time
            const int kr = u == 0 ? NXR : 0;
            if (kr > 0) {
                constexpr int XG = SPLIT && sizeof(T) > 4 ? 4 : 6;
#pragma unroll
                for (int j = 0; j < NXR / 2; ++j) asm volatile("" : "+v"(xo[j]));
                static_for<0, NXR, XG>([&](auto K0) {
                    constexpr int k0 = decltype(K0)::value;
                    if (k0 < nx) {
                        T v[XG], y[XG];
#pragma unroll
                        for (int p = 0; p < XG; ++p) {
                            y[p] = *reinterpret_cast<const T *>(
                                X + ((k0 + p) & 1 ? xo[(k0 + p) >> 1] >> 16 : xo[(k0 + p) >> 1] & 0xFFFFu));
                            v[p] = t.xv[x0 + k0 + p];
                        }
#pragma unroll
                        for (int p = 0; p < XG; ++p)
                            if (k0 + p < nx) {
                                T &o = s[SPLIT ? (k0 + p) % 4 : 0];
                                o = mad(v[p], y[p], o);
                            }
                    }
                });
            }
            for (int k = kr; k < nx; k += 4) {  // four entries' reads at a time, clamped to the row's last
                T v[4], y[4];
                uint32_t c[4];
#pragma unroll
                for (int p = 0; p < 4; ++p) {
                    const int e = x0 + (k + p < nx ? k + p : nx - 1);
                    c[p] = t.xc[e];
                    v[p] = t.xv[e];
                }
#pragma unroll
                for (int p = 0; p < 4; ++p) y[p] = *reinterpret_cast<const T *>(X + c[p]);
#pragma unroll
                for (int p = 0; p < 4; ++p)
                    if (k + p < nx) {
                        T &o = s[SPLIT ? p : 0];
                        o = mad(v[p], y[p], o);
                    }
            }
        }
        if constexpr (SPLIT) {
            acc = (s[0] + s[1]) + (s[2] + s[3]);
            bacc = (b[0] + b[1]) + (b[2] + b[3]);
        } else {
            acc = s[0];
            bacc = b[0];
        }
        __builtin_amdgcn_sched_barrier(0);
    }
};

// Forward sweep of right-hand side blockIdx.x.
template <typename T, typename OT, int RPT, bool SPLIT>
__global__ void __launch_bounds__(kSmallThreads) k_fwd_small(const SmallArgs<T> a) {
    extern __shared__ __align__(16) char lds[];
    using Rows = SmallRows<T, RPT, SPLIT, true>;
    constexpr uint32_t VB = uint32_t(Rows::CAP * sizeof(T));
    const SmallLds l = small_lds<T>(Rows::CAP, a.z, true);
    const uint32_t IB = uint32_t((l.rec - l.inc) / 2);
    uint32_t *rec = reinterpret_cast<uint32_t *>(lds + l.rec);
    T *bw = reinterpret_cast<T *>(lds + l.bw), *xv = reinterpret_cast<T *>(lds + l.xv);
    T *sw = reinterpret_cast<T *>(lds + l.sw);
    uint16_t *xc = reinterpret_cast<uint16_t *>(lds + l.xc), *sn = reinterpret_cast<uint16_t *>(lds + l.sn);
    const int tid = int(threadIdx.x), nt = int(blockDim.x), r = int(blockIdx.x);
    Rows R;
    R.load(a, rec, bw);
    for (int e = tid; e < a.z.n_x; e += nt) {
        xv[e] = a.xval[e];
        xc[e] = uint16_t(a.pos[a.xcol[e]] * int(sizeof(T)));
    }
    for (int e = tid; e < 4 * a.z.n_obs; e += nt) {
        sw[e] = a.sw[e];
        sn[e] = uint16_t(a.pos[a.snode[e]] * int(sizeof(T)));
    }
#pragma unroll
    for (int u = 0; u < RPT; ++u) {
        const int row = tid + u * nt;
        if (row < a.z.n) {
            const T v = a.in[int64_t(a.order[row]) * a.RB + r];
            reinterpret_cast<T *>(lds)[row] = v;
            reinterpret_cast<T *>(lds + 2 * VB)[row] = v;  // S^{-1} = S^0
            reinterpret_cast<T *>(lds + l.inc)[row] = v - v;
            R.own[u] = v;
            R.inc[u] = v - v;
        }
    }
    const SmallTables<T> tab{rec, bw, xv, xc, a.z.n_spec, a.z.nb4()};
    lds_barrier();
    OT *yo = static_cast<OT *>(a.y);
    const int s0 = nt - 1 - tid;  // the last threads sample: they are the ones with the fewest rows
    auto sample = [&](const char *X, const char *Y, int t) {
        if (s0 < a.z.n_obs) {
            T w[4], p[4];
            load_quad(sw + 4 * s0, w);
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const uint32_t o = sn[4 * s0 + k];
                p[k] = *reinterpret_cast<const T *>(X + o) + *reinterpret_cast<const T *>(Y + o);
            }
            T v = T(0);
#pragma unroll
            for (int k = 0; k < 4; ++k) v = mad(w[k], T(0.5) * p[k], v);
            yo[(int64_t(t) * a.z.n_obs + s0) * a.RB + r] = static_cast<OT>(static_cast<double>(v) * a.yscale);
        }
    };
    // step k: S^k in vector k % 3, S^{k-1} in (k + 2) % 3, S^{k+1} into (k + 1) % 3;
    // S^k - S^{k-1} in increment vector k % 2
    auto step = [&](auto U, int k) {
        constexpr int m = decltype(U)::value;
        const char *X = lds + m * VB, *Y = lds + (m + 2) % 3 * VB;
        const char *D = lds + l.inc + (k & 1) * IB;
        T *Z = reinterpret_cast<T *>(lds + (m + 1) % 3 * VB), *E = reinterpret_cast<T *>(lds + l.inc + (~k & 1) * IB);
        if (k > 0) sample(X, Y, k - 1);
        if (k == a.n_steps) return;
#pragma unroll
        for (int u = 0; u < RPT; ++u) {
            const int row = tid + u * nt;
            if (row < a.z.n) {
                T acc, bacc, cur;
                const T d = Rows::KEEP ? R.inc[u] : reinterpret_cast<const T *>(D)[row];
                R.template sums<false>(u, X, D, tab, acc, bacc, cur);
                const T z = step_update_d(cur, d, acc, bacc, T(0), R.dm[u], a.dt);
                Z[row] = R.own[u] = z;
                E[row] = R.inc[u] = z - cur;
            }
        }
        lds_barrier();
    };
    for (int k = 0; k <= a.n_steps; k += 3)
        static_for<0, 3>([&](auto U) {
            if (k + U.value <= a.n_steps) step(U, k + U.value);
        });
}

// Transpose sweep of right-hand side blockIdx.x.  The data of sample time t reaches the
// rows through LDS (ring slot t % 3); each sensor's thread has the loads of the next
// three sample times in flight.
template <typename T, typename YT, int RPT, bool SPLIT>
__global__ void __launch_bounds__(kSmallThreads) k_adj_small(const SmallArgs<T> a) {
    extern __shared__ __align__(16) char lds[];
    using Rows = SmallRows<T, RPT, SPLIT, false>;
    constexpr uint32_t VB = uint32_t(Rows::CAP * sizeof(T));
    const SmallLds l = small_lds<T>(Rows::CAP, a.z, false);
    const uint32_t IB = uint32_t((l.rec - l.inc) / 2);
    uint32_t *rec = reinterpret_cast<uint32_t *>(lds + l.rec);
    T *bw = reinterpret_cast<T *>(lds + l.bw), *xv = reinterpret_cast<T *>(lds + l.xv);
    T *iw = reinterpret_cast<T *>(lds + l.iw), *ring = reinterpret_cast<T *>(lds + l.ring);
    uint16_t *xc = reinterpret_cast<uint16_t *>(lds + l.xc), *is = reinterpret_cast<uint16_t *>(lds + l.is);
    const int tid = int(threadIdx.x), nt = int(blockDim.x), r = int(blockIdx.x);
    Rows R;
    R.load(a, rec, bw);
    for (int e = tid; e < a.z.n_x; e += nt) {
        xv[e] = a.xval[e];
        xc[e] = uint16_t(a.pos[a.xcol[e]] * int(sizeof(T)));
    }
    for (int e = tid; e < a.z.n_inj; e += nt) {
        iw[e] = a.injw[e];
        is[e] = uint16_t(a.injs[e]);
    }
    const int s0 = nt - 1 - tid, NT = a.n_steps;
    const bool sensor = s0 < a.z.n_obs;
    const YT *yh = static_cast<const YT *>(a.y);
    auto fetch = [&](int t) {
        return sensor && t >= 0 ? yh[(int64_t(t) * a.z.n_obs + s0) * a.RB + r] : YT(0);
    };
    auto put = [&](int t, YT v) {  // the value the step kernels read: converted to the sweep type
        if (sensor && t >= 0) ring[t % 3 * a.z.n_obs + s0] = static_cast<T>(static_cast<double>(v) * a.yscale);
    };
    // sum of the row's sensor weights times yhat^{ta} + yhat^{tb} (ta < 0: yhat^{tb})
    auto inject = [&](int u, int ta, int tb) {
        T v = T(0);
        if (!R.sp[u]) return v;
        const uint32_t re = Rows::KEEP ? R.re[u] : rec[2 * a.z.n_spec + R.sp[u] - 1];
        const int e0 = int(re & 0xFFFFu), ne = int(re >> 16);
        for (int e = e0; e < e0 + ne; ++e) {
            T d = ring[tb % 3 * a.z.n_obs + is[e]];
            if (ta >= 0) d = ring[ta % 3 * a.z.n_obs + is[e]] + d;
            v = mad(iw[e], d, v);
        }
        return v;
    };
    put(NT - 1, fetch(NT - 1));
    put(NT - 2, fetch(NT - 2));
    const SmallTables<T> tab{rec, bw, xv, xc, a.z.n_spec, a.z.nb4()};
    YT pend[3] = {fetch(NT - 3), fetch(NT - 4), fetch(NT - 5)};  // of step k in pend[k % 3]
    lds_barrier();
#pragma unroll
    for (int u = 0; u < RPT; ++u) {
        const int row = tid + u * nt;
        if (row < a.z.n) {  // q_{-1} = 0, q_0 = (dt/2m) Pi^T yhat^{N_T}
            const T v = T(0.5) * R.dm[u] * inject(u, -1, NT - 1);
            reinterpret_cast<T *>(lds)[row] = v;
            reinterpret_cast<T *>(lds + 2 * VB)[row] = T(0);
            reinterpret_cast<T *>(lds + l.inc)[row] = v;
            R.own[u] = R.inc[u] = v;
        }
    }
    lds_barrier();
    // step k: q_k in vector k % 3, q_{k-1} in (k + 2) % 3, q_{k+1} into (k + 1) % 3, q_k -
    // q_{k-1} in increment vector k % 2
    auto step = [&](auto U, int k) {
        constexpr int m = decltype(U)::value;
        const char *X = lds + m * VB, *D = lds + l.inc + (k & 1) * IB;
        T *Z = reinterpret_cast<T *>(lds + (m + 1) % 3 * VB), *E = reinterpret_cast<T *>(lds + l.inc + (~k & 1) * IB);
        const int tb = NT - 2 - k;
        put(tb - 1, pend[m]);  // read by the next step; its slot held yhat^{tb + 2}
        pend[m] = fetch(tb - 4);
#pragma unroll
        for (int u = 0; u < RPT; ++u) {
            const int row = tid + u * nt;
            if (row < a.z.n) {
                T acc, bacc, cur;
                R.template sums<false>(u, X, D, tab, acc, bacc, cur);
                const T src = T(0.5) * inject(u, tb + 1, tb);
                const T d = Rows::KEEP ? R.inc[u] : reinterpret_cast<const T *>(D)[row];
                const T z = step_update_d(cur, d, acc, bacc, src, R.dm[u], a.dt);
                Z[row] = R.own[u] = z;
                E[row] = R.inc[u] = z - cur;
            }
        }
        lds_barrier();
    };
    for (int k = 0; k < NT - 1; k += 3)
        static_for<0, 3>([&](auto U) {
            if (k + U.value < NT - 1) step(U, k + U.value);
        });
    // the closing step, with -B q_{k-1}
    const char *X = lds + (NT - 1) % 3 * VB, *Y = lds + (NT + 1) % 3 * VB;
#pragma unroll
    for (int u = 0; u < RPT; ++u) {
        const int row = tid + u * nt;
        if (row < a.z.n) {
            T acc, bacc, cur;
            R.template sums<true>(u, X, Y, tab, acc, bacc, cur);
            const T src = T(0.5) * inject(u, -1, 0), prev = reinterpret_cast<const T *>(Y)[row];
            a.out[int64_t(a.order[row]) * a.RB + r] = adj_result(cur, prev, acc, bacc, src, R.dm[u], a.dt);
        }
    }
}

SmallSizes small_sizes(const DevOps &op) {
    return SmallSizes{op.n, op.n_obs, op.n_spec, op.n_bnd, op.max_nb, op.n_x, op.n_inj};
}

template <typename T>
SmallArgs<T> small_args(const DevOps &op, int RB);
template <>
SmallArgs<double> small_args<double>(const DevOps &op, int RB) {
    return SmallArgs<double>{op.ell_col, op.xcol, op.rspec, op.order, op.pos, op.ell_val64, op.xval64, op.bslot64, op.dtm64, op.spec,
                             op.snode, op.injs, op.sw64, op.injw64, nullptr, nullptr, nullptr, 1.0,
                             small_sizes(op), op.n_steps, RB, op.dt};
}
template <>
SmallArgs<float> small_args<float>(const DevOps &op, int RB) {
    return SmallArgs<float>{op.ell_col, op.xcol, op.rspec, op.order, op.pos, op.ell_val32, op.xval32, op.bslot32, op.dtm32, op.spec,
                            op.snode, op.injs, op.sw32, op.injw32, nullptr, nullptr, nullptr, 1.0,
                            small_sizes(op), op.n_steps, RB, float(op.dt)};
}

// rows per thread, or 0 where the mesh does not fit: its rows (24 registers of float32
// or 40 of float64 operands each, of the 128 a thread of a full workgroup has), its
// tables (counts packed into 16-bit fields) or its sensors (one thread each).  Two
// float64 rows spill 9 to 42 registers in three of the four kernels and still beat the
// step launches: 1,056 / 1,690 nodes, one RHS 2.1 / 2.5 and 2.2 / 2.7 us per forward / transposed
// step against 2.7 / 2.9 and 2.9 / 3.1, 16 RHS 1.9 / 2.3 and 2.1 / 2.5 against 4.2 / 4.4 and
// 4.3 / 4.4.  (2,028 float64 nodes do not fit the LDS.)  Four float32 rows per thread would
// fit but spill, and lose: 4.4 / 5.1 against 2.9 / 3.0 us per forward / transposed step of one
// RHS on 2,940 nodes, 3.3 / 4.6 against 4.4 / 4.5 for 16.
template <typename T>
int small_rpt(const DevOps &op) {
    const int rpt = (op.n + kSmallThreads - 1) / kSmallThreads;
    if (op.n > kSmallRows || op.n_obs > kSmallThreads) return 0;
    if (op.max_nb > 16 || op.n_bnd > 0x7FFF || op.n_x > 0x7FFF || op.n_inj > 0x7FFF || op.max_spec > 0x7FFF)
        return 0;
    const SmallSizes z = small_sizes(op);
    const size_t need = std::max(small_lds<T>(rpt * kSmallThreads, z, true).total,
                                 small_lds<T>(rpt * kSmallThreads, z, false).total);
    return need <= kLdsBytes ? rpt : 0;
}

int small_threads(const DevOps &op, int rpt) {
    const int rows = ((op.n + rpt - 1) / rpt + 63) / 64 * 64, obs = (op.n_obs + 63) / 64 * 64;
    // sensors on waves of their own where the workgroup has room for them
    const int both = rows + obs;
    return both <= kSmallThreads ? both : kSmallThreads;
}

template <typename T, typename OT, int RPT, bool SPLIT>
void fwd_launch(const DevOps &op, const SmallArgs<T> &a, hipStream_t s) {
    const size_t lds = small_lds<T>(RPT * kSmallThreads, a.z, true).total;
    hipLaunchKernelGGL((k_fwd_small<T, OT, RPT, SPLIT>), dim3(a.RB), dim3(small_threads(op, RPT)), lds, s, a);
}
template <typename T, typename YT, int RPT, bool SPLIT>
void adj_launch(const DevOps &op, const SmallArgs<T> &a, hipStream_t s) {
    const size_t lds = small_lds<T>(RPT * kSmallThreads, a.z, false).total;
    hipLaunchKernelGGL((k_adj_small<T, YT, RPT, SPLIT>), dim3(a.RB), dim3(small_threads(op, RPT)), lds, s, a);
}

// rpt and the sums' order (the scalar-lane kernels' for blocks of less than 16 bytes per row)
#define PAT_SMALL(T, FN, OT, ...)                                                                      \
    do {                                                                                               \
        const bool split_ = a.RB * sizeof(T) < 16;                                                     \
        if (small_rpt<T>(op) == 1)                                                                     \
            split_ ? FN<T, OT, 1, true>(__VA_ARGS__) : FN<T, OT, 1, false>(__VA_ARGS__);               \
        else                                                                                           \
            split_ ? FN<T, OT, 2, true>(__VA_ARGS__) : FN<T, OT, 2, false>(__VA_ARGS__);               \
    } while (0)

}  // namespace

bool small_sweep_supported(Prec prec, const DevOps &op) {
    return (prec == Prec::F64 ? small_rpt<double>(op) : small_rpt<float>(op)) > 0;
}

void launch_fwd_small(Prec prec, int RB, const DevOps &op, const void *p0, void *y, bool y_is_f64, double yscale,
                      hipStream_t s) {
    if (prec == Prec::F64) {
        SmallArgs<double> a = small_args<double>(op, RB);
        a.in = static_cast<const double *>(p0);
        a.y = y;
        a.yscale = yscale;
        PAT_SMALL(double, fwd_launch, double, op, a, s);
    } else {
        SmallArgs<float> a = small_args<float>(op, RB);
        a.in = static_cast<const float *>(p0);
        a.y = y;
        a.yscale = yscale;
        if (y_is_f64) PAT_SMALL(float, fwd_launch, double, op, a, s);
        else PAT_SMALL(float, fwd_launch, float, op, a, s);
    }
}

void launch_adj_small(Prec prec, int RB, const DevOps &op, const void *yhat, bool y_is_f64, double yscale, void *out,
                      hipStream_t s) {
    if (prec == Prec::F64) {
        SmallArgs<double> a = small_args<double>(op, RB);
        a.out = static_cast<double *>(out);
        a.y = const_cast<void *>(yhat);
        a.yscale = yscale;
        PAT_SMALL(double, adj_launch, double, op, a, s);
    } else {
        SmallArgs<float> a = small_args<float>(op, RB);
        a.out = static_cast<float *>(out);
        a.y = const_cast<void *>(yhat);
        a.yscale = yscale;
        if (y_is_f64) PAT_SMALL(float, adj_launch, double, op, a, s);
        else PAT_SMALL(float, adj_launch, float, op, a, s);
    }
}

}  // namespace pat
