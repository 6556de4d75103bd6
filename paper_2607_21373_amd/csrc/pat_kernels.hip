// HIP kernels of libpat for gfx950 (MI355X, CDNA4, wave64).
//
// Data layout: a block of RB right-hand sides is stored node-major with the RHS
// fastest, x[i*RB + r], so the RB values a row gathers from one neighbour are
// one contiguous RB*sizeof(T) segment.  Blocks of at least 16 bytes per row use
// the vector-lane kernels (16 bytes per lane, further down).  Below that (one
// RHS, or two floats) the scalar-lane kernels split a row's padded slots over
// 4 lanes per RHS and combine their sums with cross-lane shuffles.
//
// Paper: "3D Uncertainty Quantification for Photoacoustic Tomography"
// (arXiv 2607.21373).  The time stepping is Sec. 3 eq. (fully-discrete) with
// M replaced by M_L; the transposed stepping is Sec. 5.1 eq. (adjoint-verlet)
// with the recursion (backward-recursion).
//
// Both are carried as three-level recurrences in one state vector, so that a
// step reads two state vectors and writes one (the velocity form reads two and
// writes two).  Forward: with S^n = p^{n+1/2} (p^{1/2} = p^0 since v^0 = 0),
// the three substeps give dt v^n = S^n - S^{n-1} and
//   S^{n+1} = S^n + (S^n - S^{n-1}) - (dt/m) (dt K S^n + B (S^n - S^{n-1})),
//   p^n = (S^{n-1} + S^n) / 2  (the sampled pressure),
// started from S^{-1} = S^0 = p^0.  Transposed: write inj_j = Pi^T yhat^{N_T - j}
// and q_k = M_L^{-1}(v_hat + dt/2 p_hat) after k transposed steps.  Then
// p_hat_{k+1} = (q_{k+1} - q_k) m/dt + B q_k + inj_{k+1}/2, and eliminating p_hat
// leaves the same recurrence for q with a source:
//   q_{k+1} = q_k + (q_k - q_{k-1}) - (dt/m) (dt K q_k + B (q_k - q_{k-1}) - (inj_k + inj_{k+1})/2)
// for k = 0 .. N_T - 2, started from q_{-1} = 0, q_0 = (dt/2m) inj_0; the result is
//   G^T yhat = (q_K - q_{K-1}) m/dt - (dt K q_K - B q_{K-1} - inj_K/2),  K = N_T - 1.
// In exact arithmetic both forms give the same maps.
#include <hip/hip_runtime.h>

#include <type_traits>

#include "pat_internal.h"
#include "pat_kernels.h"
#include "pat_step.h"
#include "pat_tiles.h"

namespace pat {
namespace {

template <int RB>
struct Geo {
    static constexpr int SPLIT = RB >= 8 ? 1 : RB == 1 ? 4 : 8 / RB;  // lanes sharing one RHS of a row
    static constexpr int LPR = RB * SPLIT;              // lanes per row
    static constexpr int RPW = 64 / LPR;                // rows per wave
    static constexpr int RPB = 4 * RPW;                 // rows per 256-thread workgroup
    static constexpr int W = 16;                        // padded slots per row (HostProblem::kEll)
    static constexpr int PER = W / SPLIT;               // padded slots per lane
};

template <int RB, int LPR>
__device__ __forceinline__ float lane_sum(float v) {
    for (int o = RB; o < LPR; o <<= 1) v += __shfl_xor(v, o);
    return v;
}
template <int RB, int LPR>
__device__ __forceinline__ double lane_sum(double v) {
    for (int o = RB; o < LPR; o <<= 1) v += __shfl_xor(v, o);
    return v;
}

// Row operands of the padded layout (see HostProblem::kEll) as the device holds it:
// slot j = p + 4 i of row r's 16 at r*16 + 4 p + i (quad p = every fourth slot), so
// that one 16-byte load gives a lane the columns (or float32 weights) of the four
// slots it sums or hands out.  Entries beyond 16 in (xptr, xcol, xval); boundary rows
// hold the B value of each slot at bslot[bsoff[row]], in the same quad order, then
// the entries beyond 16 (bsoff, xptr: a row's record).  rspec[row] is 0 for the rows with nothing but their padded
// slots, so that most rows read one word for all of that; any other row's extra ranges
// are record rspec[row] - 1 of `spec`, loaded while the first gathers are in flight.
template <typename T>
struct RowOps {
    const int32_t *ecol, *xcol;
    const T *eval, *xval, *bslot, *dtm;
    const int32_t *rspec;
    const int4 *spec;
    const int4 *rdir;  // the first half of every row's record, by row (few-wave launches)
};
// Operands of one row as seen by one lane of the scalar-lane kernels: its quad of
// padded slots (part, part + 4, ...), the row's special record and dt/m.
template <typename T, int RB>
struct RowMeta {
    int c[Geo<RB>::PER];
    T w[Geo<RB>::PER];
    int sp;
    T dm;
};

// DIRECT: launches with few waves (few_waves) wait for the record as long as for everything
// else, and read it by row with the operands, at 16 bytes a row instead of 4.
template <bool DIRECT, typename T, int RB>
__device__ __forceinline__ void load_meta(const RowOps<T> &o, int row, int part, RowMeta<T, RB> &m, RowSpec &rs) {
    using G = Geo<RB>;
    static_assert(G::SPLIT == 4 && G::PER == 4, "one quad of slots per lane");
    const int64_t eb = int64_t(row) * G::W + 4 * part;
    load_quad(o.ecol + eb, m.c);
    load_quad(o.eval + eb, m.w);
    if constexpr (DIRECT) rs.load_direct(o.rdir, row);
    else m.sp = o.rspec[row];
    m.dm = o.dtm[row];
}

// acc = sum over the row's entries of K(row, k) X[col_k][r], and for a boundary row
// bacc = sum of B(row, k) bdiff(X[col_k][r], Y[col_k][r]).  All PER gathers of the
// lane are issued before any is consumed; sums run in slot order, then the entries
// beyond 16.  rs receives the row's record (DIRECT: has it), own the row's X value (slot
// 0, in the lane of part 0).  early: loads of the caller that need the record (first) and
// what those return (second).
template <bool DIRECT, typename T, int RB, typename Early>
__device__ __forceinline__ void row_sums(const RowOps<T> &o, const RowMeta<T, RB> &m, int part, int r,
                                         const T *__restrict__ X, const T *__restrict__ Y, bool only_prev, T &acc,
                                         T &bacc, T &own, RowSpec &rs, Early &early) {
    using G = Geo<RB>;
    T x[G::PER];
#pragma unroll
    for (int j = 0; j < G::PER; ++j) x[j] = X[int64_t(m.c[j]) * RB + r];
    bool special;
    if constexpr (DIRECT) {
        special = rs.any();
    } else {
        special = m.sp != 0;
        if (special) rs.load(o.spec, m.sp);
    }
    // everything the record leads to is on its way before any of it is used; entries
    // beyond 16: XN per lane at a time, clamped to the row's last
    constexpr int XN = 3;
    int e[XN];
    uint32_t cj[XN];
    T w[XN], xv[XN], bw[G::PER], y[G::PER];
    auto fetch = [&](int k) {
#pragma unroll
        for (int j = 0; j < XN; ++j) {
            e[j] = min(k + j * G::SPLIT, rs.x1 - 1);
            cj[j] = uint32_t(o.xcol[e[j]]) * RB + r;
            w[j] = o.xval[e[j]];
        }
    };
    auto gather = [&] {
#pragma unroll
        for (int j = 0; j < XN; ++j) xv[j] = X[cj[j]];
    };
    auto add = [&](int k) {
        if (rs.nb) {
            T bv[XN], yv[XN];
#pragma unroll
            for (int j = 0; j < XN; ++j) {
                bv[j] = o.bslot[rs.bo + G::W + (e[j] - rs.x0)];
                yv[j] = Y[cj[j]];
            }
#pragma unroll
            for (int j = 0; j < XN; ++j)
                if (k + j * G::SPLIT < rs.x1) bacc = mad(bv[j], bdiff(xv[j], yv[j], only_prev), bacc);
        }
#pragma unroll
        for (int j = 0; j < XN; ++j)
            if (k + j * G::SPLIT < rs.x1) acc = mad(w[j], xv[j], acc);
    };
    int k = rs.x0 + part;
    const bool over = k < rs.x1;
    if (special) {
        if (over) fetch(k);
        early.first(rs);
        if (rs.nb) {
            load_quad(o.bslot + rs.bo + 4 * part, bw);
#pragma unroll
            for (int j = 0; j < G::PER; ++j) y[j] = Y[int64_t(m.c[j]) * RB + r];
        }
        if (over) gather();
        early.second(rs);
    }
    own = x[0];
#pragma unroll
    for (int j = 0; j < G::PER; ++j) acc = mad(m.w[j], x[j], acc);
    if (!special) return;
    if (rs.nb) {
#pragma unroll
        for (int j = 0; j < G::PER; ++j) bacc = mad(bw[j], bdiff(x[j], y[j], only_prev), bacc);
    }
    if (over) add(k);
    for (k += XN * G::SPLIT; k < rs.x1; k += XN * G::SPLIT) {
        fetch(k);
        gather();
        add(k);
    }
}

struct NothingEarly {
    __device__ __forceinline__ void first(const RowSpec &) {}
    __device__ __forceinline__ void second(const RowSpec &) {}
};

// Pi^T (yhat^{ta} + yhat^{tb}) over the injection entries of a row, for VEC right-hand sides
// from rhs0 (yhat^{ta} left out for ta < 0); A: the kernel's arguments.  The first entry's
// operands are loaded ahead of the sum if the row sums call first and second.
template <typename T, typename YT, int RB, int VEC, typename A>
struct Inject {
    const A &a;
    int rhs0;
    bool mine;  // this lane injects
    bool ahead = false;
    int s = 0;
    T w = T(0);
    YT ya[VEC], yb[VEC];
    __device__ __forceinline__ void operands(int e) {
        s = a.injs[e];
        w = a.injw[e];
    }
    __device__ __forceinline__ void data() {
        const YT *yh = static_cast<const YT *>(a.yh);
        const int64_t sb = (int64_t(a.tb) * a.n_obs + s) * RB + rhs0;
        const int64_t sa = (int64_t(a.ta) * a.n_obs + s) * RB + rhs0;
#pragma unroll
        for (int i = 0; i < VEC; ++i) yb[i] = yh[sb + i];
        if (a.ta >= 0) {
#pragma unroll
            for (int i = 0; i < VEC; ++i) ya[i] = yh[sa + i];
        }
    }
    __device__ __forceinline__ void first(const RowSpec &rs) {
        ahead = true;
        if (mine && rs.e1 > rs.e0) operands(rs.e0);
    }
    __device__ __forceinline__ void second(const RowSpec &rs) {
        if (mine && rs.e1 > rs.e0) data();
    }
    template <typename V>
    __device__ __forceinline__ void sum(const RowSpec &rs, V &&add) {
        for (int e = rs.e0; e < rs.e1; ++e) {
            if (!ahead || e > rs.e0) {
                operands(e);
                data();
            }
#pragma unroll
            for (int i = 0; i < VEC; ++i) {
                T v = static_cast<T>(static_cast<double>(yb[i]) * a.yscale);
                if (a.ta >= 0) v = static_cast<T>(static_cast<double>(ya[i]) * a.yscale) + v;
                add(i, w, v);
            }
        }
    }
};

template <typename T>
struct FwdArgs {
    RowOps<T> o;
    const int32_t *snode;
    const T *sw;
    const T *S, *Sp;  // S^n, S^{n-1}
    T *Sn;            // S^{n+1}
    void *y;
    double yscale;
    int n, n_obs, n_tiles, n_samp, sample, t;
    T dt;
};

// Forward step S^{n+1} = S^n + (S^n - S^{n-1}) - (dt/m)(dt K S^n + B (S^n - S^{n-1})),
// the three-substep Stormer-Verlet update with lumped mass in S^n = p^{n+1/2}.  One
// tile of RPB rows per workgroup; the sampling blocks placed among them write the
// samples y = Pi p^n = Pi (S^n + S^{n-1})/2 of the incoming state, one (sensor, RHS)
// pair per thread.
//
// Bound: the chain operands -> gathers -> boundary gathers of the waves on small meshes, the
// operands' traffic on large ones.  The row's own state is in hand when the sums end
// (its S^n is slot 0, its S^{n-1} comes with the operands): loaded after them it was one more
// round trip in every wave, 374,400 nodes, 1 float32 RHS 12.45 -> 11.6 us (4.8 TB/s).
template <typename T, typename OT, int RB, bool DIRECT>
__global__ void __launch_bounds__(256) k_fwd(const FwdArgs<T> a) {
    using G = Geo<RB>;
    const int tile = fwd_work(xcd_tile(blockIdx.x, gridDim.x), a.n_tiles, a.n_samp);
    if (tile < a.n_tiles) {
        const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
        const int part = (lane / RB) % G::SPLIT, r = lane % RB;
        const int row = tile * G::RPB + wave * G::RPW + lane / G::LPR;
        if (row >= a.n) return;
        RowMeta<T, RB> m;
        RowSpec rs;
        load_meta<DIRECT>(a.o, row, part, m, rs);
        const int64_t id = int64_t(row) * RB + r;
        const T prev = a.Sp[id];
        T acc = T(0), bacc = T(0), cur;
        NothingEarly none;
        row_sums<DIRECT, T, RB>(a.o, m, part, r, a.S, a.Sp, false, acc, bacc, cur, rs, none);
        acc = lane_sum<RB, G::LPR>(acc);
        bacc = lane_sum<RB, G::LPR>(bacc);
        if (part == 0) a.Sn[id] = step_update(cur, prev, acc, bacc, T(0), m.dm, a.dt);
        return;
    }
    const int64_t e = int64_t(tile - a.n_tiles) * 256 + threadIdx.x;
    if (e >= int64_t(a.n_obs) * RB) return;
    const int s = int(e / RB), r = int(e % RB);
    T y = T(0);
    for (int k = 0; k < 4; ++k) {
        const int64_t id = int64_t(a.snode[4 * s + k]) * RB + r;
        y = mad(a.sw[4 * s + k], T(0.5) * (a.S[id] + a.Sp[id]), y);
    }
    OT *yo = static_cast<OT *>(a.y);
    yo[(int64_t(a.t) * a.n_obs + s) * RB + r] = static_cast<OT>(static_cast<double>(y) * a.yscale);
}

template <typename T>
struct AdjArgs {
    RowOps<T> o;
    const int32_t *injptr, *injs;
    const T *injw;
    const T *S, *Sp;  // q_k, q_{k-1}
    T *Sn;            // q_{k+1}, or the result after the last step
    const void *yh;
    double yscale;
    int n, n_obs, n_tiles, last;
    int ta, tb;  // sources: Pi^T yhat at sample indices ta (if >= 0) and tb
    T dt;
};

// (Pi^T (yhat^{ta} + yhat^{tb}))_row for RHS r (yhat^{ta} left out for ta < 0)
template <typename T, typename YT, int RB>
__device__ __forceinline__ T inject(const AdjArgs<T> &a, int row, int r) {
    RowSpec rs;
    rs.load_inject(a.injptr, row);
    Inject<T, YT, RB, 1, AdjArgs<T>> in{a, r, true};
    T inj = T(0);
    in.sum(rs, [&](int, T w, T v) { inj = mad(w, v, inj); });
    return inj;
}

// Transposed step q_{k+1} = q_k + (q_k - q_{k-1}) - (dt/m)(dt K q_k + B (q_k - q_{k-1})
// - inj/2), inj = Pi^T (yhat^{ta} + yhat^{tb}); with `last`, the result
// (q_k - q_{k-1}) m/dt - (dt K q_k - B q_{k-1} - inj/2), inj = Pi^T yhat^{tb}.
// One tile of RPB rows per workgroup, each XCD's range walked from its end
// (xcd_tile_rev).
template <typename T, typename YT, int RB, bool DIRECT>
__global__ void __launch_bounds__(256) k_adj(const AdjArgs<T> a) {
    using G = Geo<RB>;
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const int part = (lane / RB) % G::SPLIT, r = lane % RB;
    const int wrow0 = xcd_tile_rev(blockIdx.x, gridDim.x) * G::RPB + wave * G::RPW;
    const int row = wrow0 + lane / G::LPR;
    if (row >= a.n) return;
    RowMeta<T, RB> m;
    RowSpec rs;
    load_meta<DIRECT>(a.o, row, part, m, rs);
    if constexpr (DIRECT) {
        rs.load_inject(a.injptr, row);
    }
    const int64_t id = int64_t(row) * RB + r;
    const T prev = a.Sp[id];
    T kq = T(0), bq = T(0), cur, inj = T(0);
    Inject<T, YT, RB, 1, AdjArgs<T>> in{a, r, part == 0};
    row_sums<DIRECT, T, RB>(a.o, m, part, r, a.S, a.Sp, a.last, kq, bq, cur, rs, in);
    kq = lane_sum<RB, G::LPR>(kq);
    bq = lane_sum<RB, G::LPR>(bq);
    if (part == 0) {
        in.sum(rs, [&](int, T w, T v) { inj = mad(w, v, inj); });
        const T src = T(0.5) * inj;
        a.Sn[id] = a.last ? adj_result(cur, prev, kq, bq, src, m.dm, a.dt)
                          : step_update(cur, prev, kq, bq, src, m.dm, a.dt);
    }
}

// ---------------------------------------------------------------------------
// Vector-lane step kernels (used when a row of the RHS block is >= 16 bytes).
//
// Each lane moves 16 bytes (VEC = 4 floats or 2 doubles, i.e. VEC right-hand
// sides), a lane group of LPR = RB / VEC lanes owns one row, and one wave64
// instruction gathers 64/LPR neighbour rows at once.  A row's padded operands are
// held in registers by HL = min(LPR, 4) of its lanes (each quad of lanes holds a
// copy in wider rows), loaded with 16-byte accesses and handed to the others slot
// by slot by DPP quad permutes.
//
// Bound: the chain operands -> gathers (-> boundary gathers) of each wave, then the
// traffic.  Operands staged in LDS for the whole tile (a round trip and two barriers
// more per tile, and for 16-byte rows 82 KiB of LDS per workgroup, one workgroup per
// CU) took 29.2 us per forward step of 4 float32 RHS on the 195,112-node ball against
// 9.4 us here (34 MB, 3.6 TB/s); 19.2 -> 11.9 us at 8 RHS, 19.0 -> 15.4 at 16 (63 MB,
// 4.1 TB/s), 25.5 -> 22.5 at 32; float64: 42.5 -> 12.5 us at 2 RHS, 21.5 -> 16.3 at 8.
// ---------------------------------------------------------------------------

template <typename T>
struct Vec16;
template <>
struct Vec16<float> {
    using t = float __attribute__((ext_vector_type(4)));
    static constexpr int n = 4;
};
template <>
struct Vec16<double> {
    using t = double __attribute__((ext_vector_type(2)));
    static constexpr int n = 2;
};

// Gathers in flight per lane before they are consumed.
constexpr int kGatherChunk = 8;
// Variants of the vector-lane kernels: plain, with non-temporal own rows (beyond the
// Infinity Cache), and for launches with few waves.
enum class Var : int { Plain, Stream, Few };
// Waves per SIMD the register allocation of the step kernels must allow.  Rows of 16
// or 32 bytes put 64 or 32 rows on a wave, so a launch has few waves and takes the
// registers; wider rows need the waves (two chunks of eight gathers and the four-slot
// boundary chunks fit 96 registers).
template <typename T, int RB>
constexpr int vwaves(Var v) {
    return v == Var::Few ? 2 : RB * sizeof(T) <= 32 ? 2 : 5;
}
#define PAT_VOCC(T, RB, VAR) __attribute__((amdgpu_waves_per_eu(vwaves<T, RB>(VAR))))

// Stores of the new state and loads of a row's own state (each touched once per
// step).  When the step's state exceeds the Infinity Cache (`stream`), they are
// non-temporal: caching them would only evict the neighbour rows that the gathers
// of later rows reuse, and the next step cannot find them in cache anyway.
// (A template parameter, not a run-time flag: the compiler merges two otherwise equal
// stores and drops the non-temporal hint.)
template <bool NT, typename VT, typename T>
__device__ __forceinline__ void vstore(T *p, VT v) {
    if constexpr (NT) __builtin_nontemporal_store(v, reinterpret_cast<VT *>(p));
    else *reinterpret_cast<VT *>(p) = v;
}
template <bool NT, typename VT, typename T>
__device__ __forceinline__ VT vload_own(const T *p) {
    if constexpr (NT) return __builtin_nontemporal_load(reinterpret_cast<const VT *>(p));
    else return *reinterpret_cast<const VT *>(p);
}

// Infinity Cache (memory-side last-level cache) of the MI355X
constexpr double kInfinityCacheBytes = 256.0 * 1024 * 1024;

template <typename T, int RB>
struct VGeo {
    static constexpr int VEC = Vec16<T>::n;
    static constexpr int LPR = RB / VEC;     // lanes per row
    static constexpr int RPW = 64 / LPR;     // rows per wave
    static constexpr int RPB = 4 * RPW;      // rows per 256-thread workgroup (one tile)
    static constexpr int W = 16;             // padded slots per row
    static constexpr int HL = LPR < 4 ? LPR : 4;  // lanes that share a row's padded operands
    static constexpr int QPL = 4 / HL;            // quads of slots per lane
};

// lane H of each group of HL neighbouring lanes, to the whole group (DPP quad permute;
// every lane of a group works on the same row, so none of them is ever off alone)
template <int HL, int H>
__device__ __forceinline__ uint32_t group_bcast(uint32_t x) {
    if constexpr (HL == 1) {
        return x;
    } else {
        constexpr int ctrl = HL == 4 ? H * 0x55 : H ? 0xF5 : 0xA0;
        return uint32_t(__builtin_amdgcn_update_dpp(0, int(x), ctrl, 0xF, 0xF, true));
    }
}
template <int HL, int H>
__device__ __forceinline__ int group_bcast(int x) { return int(group_bcast<HL, H>(uint32_t(x))); }
template <int HL, int H>
__device__ __forceinline__ float group_bcast(float x) {
    return __uint_as_float(group_bcast<HL, H>(__float_as_uint(x)));
}
template <int HL, int H>
__device__ __forceinline__ double group_bcast(double x) {
    const unsigned long long b = static_cast<unsigned long long>(__double_as_longlong(x));
    const unsigned long long lo = group_bcast<HL, H>(uint32_t(b)), hi = group_bcast<HL, H>(uint32_t(b >> 32));
    return __longlong_as_double(static_cast<long long>(hi << 32 | lo));
}

// v is needed here: keeps the compiler from moving its computation further down
template <typename VT>
__device__ __forceinline__ void pin(VT &v) { asm volatile("" : "+v"(v)); }

// One value per padded slot of a row, held in quads by the row's lanes (RowOps).
template <typename T, int RB, typename U>
struct SlotRegs {
    using G = VGeo<T, RB>;
    U v[4 * G::QPL];
    // lane q of the row; p: the row's 16 values in quad order
    __device__ __forceinline__ void load(const U *p, int q) {
#pragma unroll
        for (int k = 0; k < G::QPL; ++k) load_quad(p + 4 * ((q % G::HL) * G::QPL + k), v + 4 * k);
    }
    // slot J: quad J % 4, element J / 4 of it
    template <int J>
    __device__ __forceinline__ U get() const {
        constexpr int p = J % 4, i = J / 4;
        return group_bcast<G::HL, p / G::QPL>(v[4 * (p % G::QPL) + i]);
    }
};

template <typename VT, typename T>
__device__ __forceinline__ VT vfma(T w, VT x, VT acc) {
    VT o;
#pragma unroll
    for (int i = 0; i < Vec16<T>::n; ++i) o[i] = mad(w, x[i], acc[i]);
    return o;
}

// acc += sum_slots K(row, slot) X[col][q-th vector]; for boundary rows bacc +=
// B(row, slot) bdiff(X[col], Y[col]).  The B sums run after the K sums have been
// consumed, with their own gathers, so the two sets of gathers are never live
// together and the kernel keeps the register budget (and occupancy) of the interior
// rows.  Slot 0 of every row is its diagonal, so the first gather is the row's own
// X value; it is returned in `own`.  sp: the row's rspec, its record is returned in rs.
// LAT (launches with few waves, see few_waves): everything a row needs is in flight at
// once, all 16 gathers and, as soon as the row's record is there, the boundary gathers, the
// first four entries beyond the slots and the first sensor entry; the next four entries'
// operands come with each four's gathers.  An 11-entry row waits for five round trips
// instead of ten.  DIRECT: rs holds the row's record already; the transposed step does
// not take it (waiting for two tables by row costs as much as the record: 5.18 against 5.36
// us on 15,625 nodes, 16 float64 RHS).  early: as in row_sums.
template <typename T, int RB, bool LAT, bool DIRECT, typename Early>
__device__ __forceinline__ void vrow_sums(const RowOps<T> &o, int q, int sp, const T *__restrict__ X,
                                          const T *__restrict__ Y, bool only_prev, typename Vec16<T>::t &acc,
                                          typename Vec16<T>::t &bacc, typename Vec16<T>::t &own,
                                          const SlotRegs<T, RB, int> &off, const SlotRegs<T, RB, T> &kv, RowSpec &rs,
                                          Early &early) {
    using G = VGeo<T, RB>;
    using VT = typename Vec16<T>::t;
    constexpr int CH = kGatherChunk;
    // 32-bit byte offsets from the uniform bases (state arrays are < 4 GiB)
    const char *Xc = reinterpret_cast<const char *>(X);
    const char *Yc = reinterpret_cast<const char *>(Y);
    const uint32_t qoff = uint32_t(q) * 16u;
    constexpr uint32_t ROWB = uint32_t(RB * sizeof(T));
    constexpr int YL = LAT ? 12 : 0;  // boundary slots gathered early (more follow below)
    // entries beyond the padded slots, four at a time, clamped to the row's last
    int c[4];
    T w[4], w0[4];
    VT xv[4];
    auto fetch = [&](int k) {
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int e = min(k + j, rs.x1 - 1);
            c[j] = o.xcol[e];
            w[j] = o.xval[e];
        }
    };
    VT ye[YL + 1], xe[YL + 1];
    SlotRegs<T, RB, T> bv;
    if constexpr (LAT) {
        if constexpr (!DIRECT)
            if (sp) rs.load(o.spec, sp);
        VT x[G::W];
        static_for<0, G::W>([&](auto J) {
            x[J.value] = *reinterpret_cast<const VT *>(Xc + (uint32_t(off.template get<J.value>()) + qoff));
        });
        if (rs.nb) {
            bv.load(o.bslot + rs.bo, q);
            static_for<0, YL>([&](auto J) {
                ye[J.value] = *reinterpret_cast<const VT *>(Yc + (uint32_t(off.template get<J.value>()) + qoff));
            });
        }
        const bool over = rs.x1 > rs.x0;
        if (over) fetch(rs.x0);
        early.first(rs);
        if (over) {
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                xv[j] = *reinterpret_cast<const VT *>(Xc + (uint32_t(c[j]) * ROWB + qoff));
                w0[j] = w[j];
            }
            fetch(rs.x0 + 4);
        }
        early.second(rs);
        own = x[0];
        static_for<0, G::W>([&](auto J) { acc = vfma(kv.template get<J.value>(), x[J.value], acc); });
        static_for<0, YL>([&](auto J) { xe[J.value] = x[J.value]; });
#pragma unroll
        for (int j = 0; j < 4; ++j)
            if (rs.x0 + j < rs.x1) acc = vfma(w0[j], xv[j], acc);
    } else
    static_for<0, G::W, CH>([&](auto J0) {
        constexpr int j0 = decltype(J0)::value;
        VT x[CH];
        static_for<0, CH>([&](auto J) {
            constexpr int j = j0 + decltype(J)::value;
            x[J.value] = *reinterpret_cast<const VT *>(Xc + (uint32_t(off.template get<j>()) + qoff));
        });
        if constexpr (j0 == 0) {
            own = x[0];
            if (sp) rs.load(o.spec, sp);
        }
        static_for<0, CH>([&](auto J) {
            constexpr int j = j0 + decltype(J)::value;
            acc = vfma(kv.template get<j>(), x[J.value], acc);
        });
    });
    pin(acc);  // the sums end here: moved further down, they would keep the gathers live
    if (!sp) return;
    for (int k = rs.x0 + (LAT ? 4 : 0); k < rs.x1; k += 4) {
        if constexpr (!LAT) fetch(k);
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            xv[j] = *reinterpret_cast<const VT *>(Xc + (uint32_t(c[j]) * ROWB + qoff));
            w0[j] = w[j];
        }
        if constexpr (LAT) fetch(k + 4);  // the next four's operands with this four's gathers
#pragma unroll
        for (int j = 0; j < 4; ++j)
            if (k + j < rs.x1) acc = vfma(w0[j], xv[j], acc);
    }
    if (rs.nb) {
        // only the row's first bnum slots carry B; the neighbours' X values are read again
        // (the asm hides that) instead of staying live across the K sums
        uint32_t boff = qoff;
        asm volatile("" : "+v"(boff));
        const int nb = rs.nb;
        if constexpr (!LAT) bv.load(o.bslot + rs.bo, q);
        static_for<0, YL>([&](auto J) {
            VT d;
#pragma unroll
            for (int i = 0; i < G::VEC; ++i) d[i] = bdiff(xe[J.value][i], ye[J.value][i], only_prev);
            if (J.value < nb) bacc = vfma(bv.template get<J.value>(), d, bacc);
        });
        constexpr int BCH = G::HL < 4 && !LAT ? 8 : 4;  // slots at a time, two gathers each
        static_for<YL, G::W, BCH>([&](auto J0) {
            constexpr int j0 = decltype(J0)::value;
            if (j0 < nb) {
                VT y[BCH], z[BCH];
                static_for<0, BCH>([&](auto J) {
                    constexpr int j = j0 + decltype(J)::value;
                    y[J.value] = VT{};
                    z[J.value] = VT{};
                    const uint32_t at = uint32_t(off.template get<j>()) + boff;
                    if (j < nb) {
                        z[J.value] = *reinterpret_cast<const VT *>(Xc + at);
                        y[J.value] = *reinterpret_cast<const VT *>(Yc + at);
                    }
                });
                static_for<0, BCH>([&](auto J) {
                    constexpr int j = j0 + decltype(J)::value;
                    VT d;
#pragma unroll
                    for (int i = 0; i < G::VEC; ++i) d[i] = bdiff(z[J.value][i], y[J.value][i], only_prev);
                    bacc = vfma(bv.template get<j>(), d, bacc);
                });
            }
        });
        for (int k = rs.x0; k < rs.x0 + nb - G::W; ++k) {
            const uint32_t at = uint32_t(o.xcol[k]) * ROWB + qoff;
            const VT xv = *reinterpret_cast<const VT *>(Xc + at);
            const VT yv = *reinterpret_cast<const VT *>(Yc + at);
            VT dv;
#pragma unroll
            for (int i = 0; i < G::VEC; ++i) dv[i] = bdiff(xv[i], yv[i], only_prev);
            bacc = vfma(o.bslot[rs.bo + G::W + (k - rs.x0)], dv, bacc);
        }
    }
}

// The padded operands of row `row` for lane q: byte offsets of the slots' rows, and K.
template <typename T, int RB>
__device__ __forceinline__ void load_slots(const RowOps<T> &o, int row, int q, SlotRegs<T, RB, int> &off,
                                           SlotRegs<T, RB, T> &kv) {
    using G = VGeo<T, RB>;
    off.load(o.ecol + int64_t(row) * G::W, q);
    kv.load(o.eval + int64_t(row) * G::W, q);
#pragma unroll
    for (int k = 0; k < 4 * G::QPL; ++k) off.v[k] = int(uint32_t(off.v[k]) * uint32_t(RB * sizeof(T)));
}

template <typename T>
struct VFwdArgs {
    RowOps<T> o;
    const int32_t *snode;
    const T *sw;
    const T *S, *Sp;  // S^n, S^{n-1}
    T *Sn;            // S^{n+1}
    void *y;
    double yscale;
    int n, n_obs, n_tiles, n_samp, sample, t;
    int stream;  // state beyond the Infinity Cache: launch the non-temporal variant
    T dt;
};

// Sampling block j of a forward step: y = Pi (S^n + S^{n-1})/2 of the incoming
// state, one lane per (sensor, rhs).
template <typename T, typename OT, int RB>
__device__ __forceinline__ void fwd_sample(const VFwdArgs<T> &a, int j) {
    const int64_t e = int64_t(j) * 256 + threadIdx.x;
    if (e >= int64_t(a.n_obs) * RB) return;
    const int s = int(e / RB), r = int(e % RB);
    T y = T(0);
    for (int k = 0; k < 4; ++k) {
        const int64_t id = int64_t(a.snode[4 * s + k]) * RB + r;
        y = mad(a.sw[4 * s + k], T(0.5) * (a.S[id] + a.Sp[id]), y);
    }
    OT *yo = static_cast<OT *>(a.y);
    yo[(int64_t(a.t) * a.n_obs + s) * RB + r] = static_cast<OT>(static_cast<double>(y) * a.yscale);
}

// Forward step (same update as k_fwd) with vector lanes on logical tile `tile`;
// the tiles after the row tiles write the samples of the incoming state.
template <typename T, typename OT, int RB, Var VAR>
__device__ __forceinline__ void fwd_tile(const VFwdArgs<T> &a, int tile) {
    using G = VGeo<T, RB>;
    using VT = typename Vec16<T>::t;
    if (tile < a.n_tiles) {
        const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63, q = lane % G::LPR;
        const int row = tile * G::RPB + wave * G::RPW + lane / G::LPR;
        if (row >= a.n) return;
        const int64_t id = int64_t(row) * RB + q * G::VEC;
        SlotRegs<T, RB, int> off;
        SlotRegs<T, RB, T> kv;
        load_slots<T, RB>(a.o, row, q, off, kv);
        RowSpec rs;
        int sp;
        if constexpr (VAR == Var::Few) {
            rs.load_direct(a.o.rdir, row);
            sp = rs.any();
        } else {
            sp = a.o.rspec[row];
        }
        const T dm = a.o.dtm[row];
        const VT prev = vload_own<VAR == Var::Stream, VT>(a.Sp + id);
        VT acc = {}, bacc = {}, cur;
        NothingEarly none;
        vrow_sums<T, RB, VAR == Var::Few, VAR == Var::Few>(a.o, q, sp, a.S, a.Sp, false, acc, bacc, cur, off, kv, rs, none);
        VT sn;
#pragma unroll
        for (int i = 0; i < G::VEC; ++i) sn[i] = step_update(cur[i], prev[i], acc[i], bacc[i], T(0), dm, a.dt);
        vstore<VAR == Var::Stream, VT>(a.Sn + id, sn);
    } else if (a.sample) {
        fwd_sample<T, OT, RB>(a, tile - a.n_tiles);
    }
}

template <typename T, typename OT, int RB, Var VAR>
__global__ void __launch_bounds__(256) PAT_VOCC(T, RB, VAR) k_fwd_v(const VFwdArgs<T> a) {
    fwd_tile<T, OT, RB, VAR>(a, fwd_work(xcd_tile(blockIdx.x, gridDim.x), a.n_tiles, a.n_samp));
}

// Several meshes in one launch; mesh m has tiles[m] logical tiles.  Every XCD
// takes one eighth of each mesh (a contiguous range of its k-d order), as a
// launch of that mesh alone would, so each mesh's state stays spread over all
// eight L2 caches: XCD x walks, mesh after mesh, tiles
// [x q_m + min(x, r_m), +q_m + (x < r_m)) with q_m = tiles[m] / 8, r_m = tiles[m] % 8.
// The grid is 8 x the largest per-XCD count; blocks past their XCD's count idle.
template <typename A>
struct Multi {
    A a[kMaxMeshes];
    int tiles[kMaxMeshes];
    int n;
};

template <typename T, typename OT, int RB, Var VAR>
__global__ void __launch_bounds__(256) PAT_VOCC(T, RB, VAR) k_fwd_vm(const Multi<VFwdArgs<T>> mm) {
    int m, local;
    if (!mesh_tile(mm.tiles, mm.n, blockIdx.x, &m, &local, false)) return;
    fwd_tile<T, OT, RB, VAR>(mm.a[m], fwd_work(local, mm.a[m].n_tiles, mm.a[m].n_samp));
}

template <typename T>
struct VAdjArgs {
    RowOps<T> o;
    const int32_t *injs;
    const T *injw;
    const T *S, *Sp;  // q_k, q_{k-1}
    T *Sn;            // q_{k+1}, or the result after the last step
    const void *yh;
    double yscale;
    int n, n_obs, n_tiles, last;
    int ta, tb;  // sources: Pi^T yhat at sample indices ta (if >= 0) and tb
    int stream;  // state beyond the Infinity Cache: launch the non-temporal variant
    T dt;
};

// Transposed step (same update as k_adj) with vector lanes on logical tile `tile`;
// LAST: the closing launch.
template <typename T, typename YT, int RB, Var VAR, bool LAST>
__device__ __forceinline__ void adj_tile(const VAdjArgs<T> &a, int tile) {
    using G = VGeo<T, RB>;
    using VT = typename Vec16<T>::t;
    if (tile >= a.n_tiles) return;
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63, q = lane % G::LPR;
    const int row = tile * G::RPB + wave * G::RPW + lane / G::LPR;
    if (row >= a.n) return;
    const int64_t id = int64_t(row) * RB + q * G::VEC;
    RowSpec rs;
    const int sp = a.o.rspec[row];
    SlotRegs<T, RB, int> off;
    SlotRegs<T, RB, T> kv;
    load_slots<T, RB>(a.o, row, q, off, kv);
    const T dm = a.o.dtm[row];
    const VT prev = vload_own<VAR == Var::Stream, VT>(a.Sp + id);
    VT kq = {}, bq = {}, cur, inj = {};
    Inject<T, YT, RB, G::VEC, VAdjArgs<T>> in{a, q * G::VEC, true};
    vrow_sums<T, RB, VAR == Var::Few, false>(a.o, q, sp, a.S, a.Sp, LAST, kq, bq, cur, off, kv, rs, in);
    in.sum(rs, [&](int i, T w, T v) { inj[i] = mad(w, v, inj[i]); });
    VT out;
#pragma unroll
    for (int i = 0; i < G::VEC; ++i) {
        const T src = T(0.5) * inj[i];
        if constexpr (LAST) out[i] = adj_result(cur[i], prev[i], kq[i], bq[i], src, dm, a.dt);
        else out[i] = step_update(cur[i], prev[i], kq[i], bq[i], src, dm, a.dt);
    }
    vstore<VAR == Var::Stream, VT>(a.Sn + id, out);
}

template <typename T, typename YT, int RB, Var VAR, bool LAST>
__global__ void __launch_bounds__(256) PAT_VOCC(T, RB, VAR) k_adj_v(const VAdjArgs<T> a) {
    adj_tile<T, YT, RB, VAR, LAST>(a, xcd_tile_rev(blockIdx.x, gridDim.x));
}

template <typename T, typename YT, int RB, Var VAR, bool LAST>
__global__ void __launch_bounds__(256) PAT_VOCC(T, RB, VAR) k_adj_vm(const Multi<VAdjArgs<T>> mm) {
    int m, local;
    if (!mesh_tile(mm.tiles, mm.n, blockIdx.x, &m, &local, true)) return;
    adj_tile<T, YT, RB, VAR, LAST>(mm.a[m], local);
}

// q_{-1} = 0 and q_0 = (dt/2m) Pi^T yhat^{tb} (tb = N_T - 1, the last sample)
template <typename T, typename YT, int RB>
__global__ void __launch_bounds__(256) k_adj_init(const AdjArgs<T> a, T *q0, T *qm1) {
    const int64_t total = int64_t(a.n) * RB;
    for (int64_t e = int64_t(blockIdx.x) * 256 + threadIdx.x; e < total; e += int64_t(gridDim.x) * 256) {
        const int row = int(e / RB), r = int(e % RB);
        q0[e] = T(0.5) * a.o.dtm[row] * inject<T, YT, RB>(a, row, r);
        qm1[e] = T(0);
    }
}

// ---------------------------------------------------------------------------
// Layout conversions (LDS-tiled transposes)
// ---------------------------------------------------------------------------

// out[c][r] = in[rb0 + r][perm(c)] (zero for rb0 + r >= R), tile of 64 columns x 64 RHS,
// the block's RHS in chunks of 64
template <typename TI, typename TO>
__global__ void __launch_bounds__(256) k_pack(const TI *in, int64_t R, int64_t rb0, int RB, int64_t cols,
                                              const int32_t *perm, TO *out) {
    __shared__ double tile[64][65];
    const int64_t c0 = int64_t(blockIdx.x) * 64;
    for (int r0 = 0; r0 < RB; r0 += 64) {
        const int rn = RB - r0 < 64 ? RB - r0 : 64;
        for (int e = threadIdx.x; e < 64 * rn; e += 256) {
            const int r = e / 64, c = e % 64;
            const int64_t cc = c0 + c, rr = rb0 + r0 + r;
            double v = 0.0;
            if (cc < cols && rr < R) v = static_cast<double>(in[rr * cols + (perm ? perm[cc] : cc)]);
            tile[r][c] = v;
        }
        __syncthreads();
        for (int e = threadIdx.x; e < 64 * rn; e += 256) {
            const int c = e / rn, r = e % rn;
            const int64_t cc = c0 + c;
            if (cc < cols) out[cc * RB + r0 + r] = static_cast<TO>(tile[r][c]);
        }
        __syncthreads();
    }
}

// out[rb0 + r][perm(c)] = in[c][r] for rb0 + r < R (same tiling as k_pack)
template <typename TI, typename TO>
__global__ void __launch_bounds__(256) k_unpack(const TI *in, int64_t R, int64_t rb0, int RB, int64_t cols,
                                                const int32_t *perm, TO *out) {
    __shared__ double tile[64][65];
    const int64_t c0 = int64_t(blockIdx.x) * 64;
    for (int r0 = 0; r0 < RB; r0 += 64) {
        const int rn = RB - r0 < 64 ? RB - r0 : 64;
        for (int e = threadIdx.x; e < 64 * rn; e += 256) {
            const int c = e / rn, r = e % rn;
            const int64_t cc = c0 + c;
            tile[r][c] = cc < cols ? static_cast<double>(in[cc * RB + r0 + r]) : 0.0;
        }
        __syncthreads();
        for (int e = threadIdx.x; e < 64 * rn; e += 256) {
            const int r = e / 64, c = e % 64;
            const int64_t cc = c0 + c, rr = rb0 + r0 + r;
            if (cc < cols && rr < R) out[rr * cols + (perm ? perm[cc] : cc)] = static_cast<TO>(tile[r][c]);
        }
        __syncthreads();
    }
}

// ---- counter-based standard normals -------------------------------------
// Philox4x64-10 (Salmon et al., SC'11) and the Box-Muller transform.  Normal j
// of stream (seed, kind, k) is lane j%4 of the cipher block with counter
// (j/4, k, kind, 0) and key (seed, 0); lanes (0,1) and (2,3) are Box-Muller
// pairs with u1 = 1 - U(w_even) in (0, 1], u2 = U(w_odd), U(w) = (w >> 11) 2^-53.
struct Normals4 {
    double z[4];
};

__device__ inline Normals4 philox_normals(uint64_t seed, uint64_t kind, uint64_t k, uint64_t blk) {
    uint64_t c0 = blk, c1 = k, c2 = kind, c3 = 0, k0 = seed, k1 = 0;
#pragma unroll
    for (int round = 0; round < 10; ++round) {
        if (round > 0) {
            k0 += 0x9E3779B97F4A7C15ULL;
            k1 += 0xBB67AE8584CAA73BULL;
        }
        const uint64_t hi0 = __umul64hi(0xD2E7470EE14C6C93ULL, c0), lo0 = 0xD2E7470EE14C6C93ULL * c0;
        const uint64_t hi1 = __umul64hi(0xCA5A826395121157ULL, c2), lo1 = 0xCA5A826395121157ULL * c2;
        c0 = hi1 ^ c1 ^ k0;
        c1 = lo1;
        c2 = hi0 ^ c3 ^ k1;
        c3 = lo0;
    }
    Normals4 o;
    const uint64_t w[4] = {c0, c1, c2, c3};
#pragma unroll
    for (int pr = 0; pr < 2; ++pr) {
        const double u1 = 1.0 - double(w[2 * pr] >> 11) * 0x1p-53;
        const double u2 = double(w[2 * pr + 1] >> 11) * 0x1p-53;
        const double rad = sqrt(-2.0 * log(u1));
        const double ang = 6.283185307179586476925286766559 * u2;
        o.z[2 * pr] = rad * cos(ang);
        o.z[2 * pr + 1] = rad * sin(ang);
    }
    return o;
}

// out[s*len + j] = normal j of stream (seed, kind, k0 + s)
__global__ void __launch_bounds__(256) k_normals(uint64_t seed, int kind, int64_t k0, int64_t S, int64_t len,
                                                 double *out) {
    const int64_t nblk = (len + 3) / 4, total = S * nblk;
    for (int64_t e = int64_t(blockIdx.x) * blockDim.x + threadIdx.x; e < total; e += int64_t(gridDim.x) * blockDim.x) {
        const int64_t sm = e / nblk, b = e % nblk;
        const Normals4 z = philox_normals(seed, uint64_t(kind), uint64_t(k0 + sm), uint64_t(b));
#pragma unroll
        for (int l = 0; l < 4; ++l)
            if (4 * b + l < len) out[sm * len + 4 * b + l] = z.z[l];
    }
}

// bd[m][r] = yobs[m] * isig + eta_{k0+rb0+r}[m] drawn on the fly (zero rows past S)
__global__ void __launch_bounds__(256) k_build_rhs_rng(const double *yobs, uint64_t seed, int64_t k0, int64_t S,
                                                       int64_t rb0, int RB, int64_t M, double isig, double *bd) {
    const int64_t nblk = (M + 3) / 4, total = nblk * RB;
    for (int64_t e = int64_t(blockIdx.x) * blockDim.x + threadIdx.x; e < total; e += int64_t(gridDim.x) * blockDim.x) {
        const int64_t b = e / RB;
        const int r = int(e % RB);
        const bool live = rb0 + r < S;
        Normals4 z{};
        if (live) z = philox_normals(seed, 0, uint64_t(k0 + rb0 + r), uint64_t(b));
#pragma unroll
        for (int l = 0; l < 4; ++l) {
            const int64_t m = 4 * b + l;
            if (m < M) bd[m * RB + r] = live ? yobs[m] * isig + z.z[l] : 0.0;
        }
    }
}

// xi[q][r] = normal perm(q) of stream (seed, 1, k0+rb0+r), internal node order (zero rows past S)
__global__ void __launch_bounds__(256) k_xi_rng(uint64_t seed, int64_t k0, int64_t S, int64_t rb0, int RB, int64_t N,
                                                const int32_t *perm, double *xi) {
    const int64_t total = N * RB;
    for (int64_t e = int64_t(blockIdx.x) * blockDim.x + threadIdx.x; e < total; e += int64_t(gridDim.x) * blockDim.x) {
        const int64_t q = e / RB;
        const int r = int(e % RB);
        double v = 0.0;
        if (rb0 + r < S) {
            const int64_t j = perm ? perm[q] : q;
            v = philox_normals(seed, 1, uint64_t(k0 + rb0 + r), uint64_t(j / 4)).z[j % 4];
        }
        xi[e] = v;
    }
}

// bd[m][r] = yobs[m] * isig + eta[rb0 + r][m]  (zero rows past S); RHS in chunks of 64
__global__ void __launch_bounds__(256) k_build_rhs(const double *yobs, const double *eta, int64_t S, int64_t rb0,
                                                   int RB, int64_t M, double isig, double *bd) {
    __shared__ double tile[64][65];
    const int64_t c0 = int64_t(blockIdx.x) * 64;
    for (int r0 = 0; r0 < RB; r0 += 64) {
        const int rn = RB - r0 < 64 ? RB - r0 : 64;
        for (int e = threadIdx.x; e < 64 * rn; e += 256) {
            const int r = e / 64, c = e % 64;
            const int64_t cc = c0 + c, rr = rb0 + r0 + r;
            tile[r][c] = (cc < M && rr < S) ? eta[rr * M + cc] : 0.0;
        }
        __syncthreads();
        for (int e = threadIdx.x; e < 64 * rn; e += 256) {
            const int c = e / rn, r = e % rn;
            const int64_t cc = c0 + c;
            if (cc < M) bd[cc * RB + r0 + r] = (rb0 + r0 + r < S) ? yobs[cc] * isig + tile[r][c] : 0.0;
        }
        __syncthreads();
    }
}

// ---------------------------------------------------------------------------
// CGLS helpers (float64)
// ---------------------------------------------------------------------------

__global__ void k_fill(double *x, int64_t n, double v) {
    for (int64_t e = int64_t(blockIdx.x) * blockDim.x + threadIdx.x; e < n; e += int64_t(gridDim.x) * blockDim.x) x[e] = v;
}

template <typename T>
__global__ void k_cast(const double *x, T *y, int64_t n) {
    for (int64_t e = int64_t(blockIdx.x) * blockDim.x + threadIdx.x; e < n; e += int64_t(gridDim.x) * blockDim.x)
        y[e] = static_cast<T>(x[e]);
}

// y = L x = M_L^{1/2} x + a M_L^{-1/2} (K1 x)
// float64 value of lane l of v (l wave-uniform)
__device__ __forceinline__ double readlane_f64(double v, int l) {
    const long long b = __double_as_longlong(v);
    const unsigned lo = unsigned(__builtin_amdgcn_readlane(int(b), l));
    const unsigned hi = unsigned(__builtin_amdgcn_readlane(int(b >> 32), l));
    return __longlong_as_double(static_cast<long long>((static_cast<unsigned long long>(hi) << 32) | lo));
}

// sum over the entries k of row i of the K1 pattern, in ascending order, of
// fma(K1[k], f_j x[j RB + r], acc) with j = col[k] and f_j = isqrtm[j] (SCALE) or
// the plain x value, for a wave-uniform row i (RB >= 64, one row per wave): lane l
// holds entry k0 + l's column, value and scale, read back by readlane, and the
// gathers go in groups of 16, all issued before the first is used (the same sums
// as entry by entry, in the same order, with a few dependent round trips per row
// instead of one per entry)
template <bool SCALE>
__device__ __forceinline__ double k1_row_wave(const int32_t *rowptr, const int32_t *col, const double *k1,
                                             const double *isqrtm, int i, int RB, int r, const double *x) {
    constexpr int G = 16;
    const int lane = int(threadIdx.x) & 63;
    const int k0 = rowptr[i], ke = rowptr[i + 1];
    double acc = 0.0;
    for (int kb = k0; kb < ke; kb += 64) {
        const int nk = min(64, ke - kb);
        int cl = 0;
        double wl = 0.0, sl = 1.0;
        if (lane < nk) {
            cl = col[kb + lane];
            wl = k1[kb + lane];
            if (SCALE) sl = isqrtm[cl];
        }
        for (int g = 0; g < nk; g += G) {
            double xv[G];
#pragma unroll
            for (int j = 0; j < G; ++j)  // past the end: the last entry again, loaded but not summed
                xv[j] = x[int64_t(__builtin_amdgcn_readlane(cl, min(g + j, nk - 1))) * RB + r];
#pragma unroll
            for (int j = 0; j < G; ++j)
                if (g + j < nk) {
                    const double w = readlane_f64(wl, g + j);
                    acc = SCALE ? __builtin_fma(w, readlane_f64(sl, g + j) * xv[j], acc) : __builtin_fma(w, xv[j], acc);
                }
        }
    }
    return acc;
}

__global__ void __launch_bounds__(256) k_prior(const int32_t *rowptr, const int32_t *col, const double *k1,
                                               const double *sqrtm, const double *isqrtm, int n, int RB, double a,
                                               const double *x, double *y) {
    // 256 / RB rows per block and pass, thread (row lr, RHS r); with RB >= 64 a wave
    // holds one row, whose operands are then wave-uniform (scalar loads)
    const int rpb = 256 / RB, r = int(threadIdx.x) % RB, lr = int(threadIdx.x) / RB;
    auto row = [&](int i, bool wave_row) {
        double acc = 0.0;
        if (wave_row) {
            acc = k1_row_wave<false>(rowptr, col, k1, isqrtm, i, RB, r, x);
        } else {
#pragma unroll 4
            for (int k = rowptr[i]; k < rowptr[i + 1]; ++k) acc = __builtin_fma(k1[k], x[int64_t(col[k]) * RB + r], acc);
        }
        const int64_t e = int64_t(i) * RB + r;
        y[e] = sqrtm[i] * x[e] + a * isqrtm[i] * acc;
    };
    for (int64_t i = int64_t(blockIdx.x) * rpb + lr; i < n; i += int64_t(gridDim.x) * rpb) {
        if (RB >= 64) row(__builtin_amdgcn_readfirstlane(int(i)), true);
        else row(int(i), false);
    }
}

// out = isig * PH + L^T rp,  L^T rp = M_L^{1/2} rp + a K1 (M_L^{-1/2} rp); PH is the
// transpose sweep's result G^T r_d
template <typename T>
__global__ void __launch_bounds__(256) k_gext_t(const int32_t *rowptr, const int32_t *col, const double *k1,
                                                const double *sqrtm, const double *isqrtm, int n, int RB, double a,
                                                double isig, const T *PH, const double *rp, double *out) {
    // as k_prior: 256 / RB rows per block and pass; wave-uniform rows for RB >= 64
    const int rpb = 256 / RB, r = int(threadIdx.x) % RB, lr = int(threadIdx.x) / RB;
    auto row = [&](int i, bool wave_row) {
        double acc = 0.0;
        if (wave_row) {
            acc = k1_row_wave<true>(rowptr, col, k1, isqrtm, i, RB, r, rp);
        } else {
#pragma unroll 4
            for (int k = rowptr[i]; k < rowptr[i + 1]; ++k) {
                const int j = col[k];
                acc = __builtin_fma(k1[k], isqrtm[j] * rp[int64_t(j) * RB + r], acc);
            }
        }
        const int64_t e = int64_t(i) * RB + r;
        out[e] = isig * static_cast<double>(PH[e]) + (sqrtm[i] * rp[e] + a * acc);
    };
    for (int64_t i = int64_t(blockIdx.x) * rpb + lr; i < n; i += int64_t(gridDim.x) * rpb) {
        if (RB >= 64) row(__builtin_amdgcn_readfirstlane(int(i)), true);
        else row(int(i), false);
    }
}

// y = L^T x = M_L^{1/2} x + a K1 (M_L^{-1/2} x)
__global__ void __launch_bounds__(256) k_prior_t(const int32_t *rowptr, const int32_t *col, const double *k1,
                                                 const double *sqrtm, const double *isqrtm, int n, int RB, double a,
                                                 const double *x, double *y) {
    // as k_prior: 256 / RB rows per block and pass; wave-uniform rows for RB >= 64
    const int rpb = 256 / RB, r = int(threadIdx.x) % RB, lr = int(threadIdx.x) / RB;
    auto row = [&](int i, bool wave_row) {
        double acc = 0.0;
        if (wave_row) {
            acc = k1_row_wave<true>(rowptr, col, k1, isqrtm, i, RB, r, x);
        } else {
#pragma unroll 4
            for (int k = rowptr[i]; k < rowptr[i + 1]; ++k) {
                const int j = col[k];
                acc = __builtin_fma(k1[k], isqrtm[j] * x[int64_t(j) * RB + r], acc);
            }
        }
        const int64_t e = int64_t(i) * RB + r;
        y[e] = sqrtm[i] * x[e] + a * acc;
    };
    for (int64_t i = int64_t(blockIdx.x) * rpb + lr; i < n; i += int64_t(gridDim.x) * rpb) {
        if (RB >= 64) row(__builtin_amdgcn_readfirstlane(int(i)), true);
        else row(int(i), false);
    }
}

// Squares of x [rows][RB] summed over the rows of block b of nb into part[b][r].  Four rows
// per pass into four partial sums, so that each lane keeps four loads in flight.
__device__ __forceinline__ void norm_partial(const double *x, int64_t rows, int RB, int b, int nb, double *part,
                                             double *red) {
    const int G = 256 / RB;
    const int r = threadIdx.x % RB, g = threadIdx.x / RB;
    const int64_t chunk = (rows + nb - 1) / nb;
    const int64_t a0 = int64_t(b) * chunk, a1 = a0 + chunk < rows ? a0 + chunk : rows;
    double acc0 = 0.0, acc1 = 0.0, acc2 = 0.0, acc3 = 0.0;
    int64_t row = a0 + g;
    for (; row + 3 * G < a1; row += 4 * G) {
        const double v0 = x[row * RB + r], v1 = x[(row + G) * RB + r], v2 = x[(row + 2 * G) * RB + r],
                     v3 = x[(row + 3 * G) * RB + r];
        acc0 = __builtin_fma(v0, v0, acc0);
        acc1 = __builtin_fma(v1, v1, acc1);
        acc2 = __builtin_fma(v2, v2, acc2);
        acc3 = __builtin_fma(v3, v3, acc3);
    }
    for (; row < a1; row += G) {
        const double v = x[row * RB + r];
        acc0 = __builtin_fma(v, v, acc0);
    }
    red[threadIdx.x] = (acc0 + acc1) + (acc2 + acc3);
    __syncthreads();
    for (int s = 128; s >= RB; s >>= 1) {
        if (threadIdx.x < s) red[threadIdx.x] += red[threadIdx.x + s];
        __syncthreads();
    }
    if (threadIdx.x < RB) part[int64_t(b) * RB + threadIdx.x] = red[threadIdx.x];
}

// The partial norms of one or two arrays in one launch: na blocks on x, nb on y.  Each
// scalar stage below finishes the norms it needs in its own launch: on small meshes a solver
// iteration is a chain of 5 us launches (4913 nodes, 200 steps, 16 float32 samples,
// 50 LSQR iterations: 115 -> 101 ms with the reductions of this file; 864 nodes, 10 float64
// samples, 30 CGLS iterations: 28.0 -> 23.9 ms).
__global__ void __launch_bounds__(256) k_norms(const double *x, int64_t xrows, int na, double *pa, const double *y,
                                               int64_t yrows, int nb, double *pb, int RB) {
    __shared__ double red[256];
    const int b = int(blockIdx.x);
    if (b < na) norm_partial(x, xrows, RB, b, na, pa, red);
    else norm_partial(y, yrows, RB, b - na, nb, pb, red);
}

// part[b][r] = sum over rows of block b of (a[row][aoff + r] - y[row][r])^2, a with row
// stride lda, y with row stride RB (the reduction tree of norm_partial)
__global__ void __launch_bounds__(256) k_diff_sq_partial(const double *a, int lda, int aoff, const double *y,
                                                         int64_t rows, int RB, double *part) {
    __shared__ double red[256];
    const int G = 256 / RB;
    const int r = threadIdx.x % RB, g = threadIdx.x / RB;
    const int64_t chunk = (rows + gridDim.x - 1) / gridDim.x;
    const int64_t a0 = int64_t(blockIdx.x) * chunk, a1 = a0 + chunk < rows ? a0 + chunk : rows;
    double acc = 0.0;
    for (int64_t row = a0 + g; row < a1; row += G) {
        const double d = a[row * lda + aoff + r] - y[row * RB + r];
        acc = __builtin_fma(d, d, acc);
    }
    red[threadIdx.x] = acc;
    __syncthreads();
    for (int s = 128; s >= RB; s >>= 1) {
        if (threadIdx.x < s) red[threadIdx.x] += red[threadIdx.x + s];
        __syncthreads();
    }
    if (threadIdx.x < RB) part[int64_t(blockIdx.x) * RB + threadIdx.x] = red[threadIdx.x];
}

// out[row][r] = in[row][c0 + r], r < RB (in with row stride ldin)
__global__ void k_cols(const double *in, int ldin, int c0, double *out, int64_t total, int RB) {
    for (int64_t e = int64_t(blockIdx.x) * blockDim.x + threadIdx.x; e < total; e += int64_t(gridDim.x) * blockDim.x)
        out[e] = in[(e / RB) * ldin + c0 + e % RB];
}

// acc + p[b0 stride] + p[(b0 + G) stride] + ... in that order, 16 loads at a time: one
// workgroup sums all partial blocks, and its loads' latency is what it costs.
__device__ __forceinline__ double strided_sum(const double *p, int b, int G, int nb, int64_t stride, double acc) {
    for (; b + 15 * G < nb; b += 16 * G) {
        double v[16];
#pragma unroll
        for (int q = 0; q < 16; ++q) v[q] = p[int64_t(b + q * G) * stride];
#pragma unroll
        for (int q = 0; q < 16; ++q) acc += v[q];
    }
    for (; b < nb; b += G) acc += p[int64_t(b) * stride];
    return acc;
}

// sum over the na blocks of pa (and then the nb of pb), for thread r < RB of the workgroup
__device__ __forceinline__ double sum_parts(const double *pa, int na, const double *pb, int nb, int RB, double *red) {
    const int G = 256 / RB;
    const int r = threadIdx.x % RB, g = threadIdx.x / RB;
    double acc = strided_sum(pa + r, g, G, na, RB, 0.0);
    if (pb) acc = strided_sum(pb + r, g, G, nb, RB, acc);
    __syncthreads();
    red[threadIdx.x] = acc;
    __syncthreads();
    for (int s = 128; s >= RB; s >>= 1) {
        if (threadIdx.x < s) red[threadIdx.x] += red[threadIdx.x + s];
        __syncthreads();
    }
    return red[r];
}

__global__ void __launch_bounds__(256) k_norm_store(const NormParts n, int RB, double *out) {
    __shared__ double red[256];
    const double v = sum_parts(n.a, n.na, n.b, n.nb, RB, red);
    if (threadIdx.x < RB) out[threadIdx.x] = v;
}

// alpha = gamma / ||(x, y)||^2
__global__ void __launch_bounds__(256) k_norm_alpha(const NormParts n, int RB, const double *gamma, double *alpha) {
    __shared__ double red[256];
    const double delta = sum_parts(n.a, n.na, n.b, n.nb, RB, red);
    const int r = threadIdx.x;
    if (r < RB) alpha[r] = delta > 0.0 ? gamma[r] / delta : 0.0;
}

// g = ||x||^2: beta = g / gamma, invn = 1 / ||x||, gamma = g
__global__ void __launch_bounds__(256) k_norm_gamma(const NormParts n, int RB, double *gamma, double *beta,
                                                    double *invn, int first) {
    __shared__ double red[256];
    const double g = sum_parts(n.a, n.na, n.b, n.nb, RB, red);
    const int r = threadIdx.x;
    if (r >= RB) return;
    beta[r] = (first || !(gamma[r] > 0.0)) ? 0.0 : g / gamma[r];
    invn[r] = g > 0.0 ? 1.0 / sqrt(g) : 0.0;
    gamma[r] = g;
}

// hist and diag of one right-hand side from its squared data and prior residuals
__device__ __forceinline__ void store_resid(double a, double b, double *hist, double *diag, int64_t at) {
    if (hist) hist[at] = sqrt(a + b);
    if (diag) {
        diag[2 * at] = sqrt(a);
        diag[2 * at + 1] = sqrt(b);
    }
}

__global__ void __launch_bounds__(256) k_norm_resid(const NormParts n, int RB, double *hist, double *diag, int64_t ld,
                                                    int64_t col, int64_t rb0, int64_t R) {
    __shared__ double red[256];
    const double a = sum_parts(n.a, n.na, nullptr, 0, RB, red), b = sum_parts(n.b, n.nb, nullptr, 0, RB, red);
    const int r = threadIdx.x;
    if (r < RB && rb0 + r < R) store_resid(a, b, hist, diag, (rb0 + r) * ld + col);
}

__global__ void k_resid(const double *a, const double *b, double *hist, double *diag, int64_t ld, int64_t col,
                        int64_t rb0, int64_t R, int RB) {
    const int r = threadIdx.x;
    if (r < RB && rb0 + r < R) store_resid(a[r], b[r], hist, diag, (rb0 + r) * ld + col);
}

// Grid-stride loops over [rows][RB] arrays: the RHS index of a thread's elements,
// fixed when the stride is a multiple of RB (RB a power of two <= the block size),
// so that no element pays a 64-bit division.
struct RhsIndex {
    int64_t stride;
    int r0, RB;
    bool fixed;
    __device__ RhsIndex(int rb) : RB(rb) {
        stride = int64_t(gridDim.x) * blockDim.x;
        r0 = int((int64_t(blockIdx.x) * blockDim.x + threadIdx.x) % rb);
        fixed = stride % rb == 0;
    }
    __device__ int operator()(int64_t e) const { return fixed ? r0 : int(e % RB); }
};

__global__ void k_update_xr(double *x, const double *d, double *rp, const double *qp, const double *alpha,
                            int64_t total, int RB) {
    const RhsIndex rix(RB);
    for (int64_t e = int64_t(blockIdx.x) * blockDim.x + threadIdx.x; e < total; e += rix.stride) {
        const double al = alpha[rix(e)];
        x[e] += al * d[e];
        rp[e] -= al * qp[e];
    }
}

__global__ void k_axpy_neg(double *y, const double *x, const double *alpha, int64_t total, int RB) {
    const RhsIndex rix(RB);
    for (int64_t e = int64_t(blockIdx.x) * blockDim.x + threadIdx.x; e < total; e += rix.stride)
        y[e] -= alpha[rix(e)] * x[e];
}

__global__ void k_append(const double *sv, double *Qk, double *d, const double *invn, const double *beta, int first,
                         int64_t total, int RB) {
    const RhsIndex rix(RB);
    for (int64_t e = int64_t(blockIdx.x) * blockDim.x + threadIdx.x; e < total; e += rix.stride) {
        const int r = rix(e);
        const double s = sv[e];
        if (Qk) Qk[e] = s * invn[r];
        d[e] = first ? s : s + beta[r] * d[e];
    }
}

// ---- LSQR (Golub-Kahan bidiagonalisation) ---------------------------------
// Per-RHS scalar stages; one thread per right-hand side.  A new alpha or beta
// below 1e-15 of its first value is exact breakdown and is set to zero.
__global__ void __launch_bounds__(256) k_lsqr_scalar(LsqrStage st, LsqrScalars c, const NormParts n, int RB) {
    __shared__ double red[256];
    const double n1 = sum_parts(n.a, n.na, nullptr, 0, RB, red);
    const double n2 = n.b ? sum_parts(n.b, n.nb, nullptr, 0, RB, red) : 0.0;
    const int r = threadIdx.x;
    if (r >= RB) return;
    const double nrm = sqrt(n1 + n2);
    switch (st) {
    case LsqrStage::InitBeta:
        c.beta[r] = c.beta1[r] = nrm;
        c.inv[r] = nrm > 0.0 ? 1.0 / nrm : 0.0;
        break;
    case LsqrStage::InitAlpha:
        c.alpha[r] = c.alpha1[r] = nrm;
        c.inv[r] = nrm > 0.0 ? 1.0 / nrm : 0.0;
        c.phib[r] = c.beta[r];
        c.rhob[r] = nrm;
        c.zfac[r] = 0.0;
        break;
    case LsqrStage::Beta: {
        const double be = nrm > 1e-15 * c.beta1[r] ? nrm : 0.0;
        c.beta[r] = be;
        c.inv[r] = be > 0.0 ? 1.0 / be : 0.0;
        // plane rotation eliminating beta_{k+1} below rho_bar_k
        const double rb = c.rhob[r];
        const double rho = sqrt(rb * rb + be * be);
        const double cs = rho > 0.0 ? rb / rho : 1.0, sn = rho > 0.0 ? be / rho : 0.0;
        const double phi = cs * c.phib[r];
        c.rho[r] = rho;
        c.cs[r] = cs;
        c.sn[r] = sn;
        c.phib[r] = sn * c.phib[r];
        c.step[r] = rho > 0.0 ? phi / rho : 0.0;
        break;
    }
    case LsqrStage::Alpha: {
        const double al = nrm > 1e-15 * c.alpha1[r] ? nrm : 0.0;
        c.alpha[r] = al;
        c.inv[r] = al > 0.0 ? 1.0 / al : 0.0;
        c.rhob[r] = -c.cs[r] * al;
        c.zfac[r] = c.rho[r] > 0.0 ? c.sn[r] * al / c.rho[r] : 0.0;
        break;
    }
    }
}

// out = (sa * ca[r]) a + (sb * cb[r]) b; a null coefficient pointer means 1, b may be null.
__global__ void k_lincomb(double *out, const double *a, const double *ca, double sa, const double *b, const double *cb,
                          double sb, int64_t total, int RB) {
    const RhsIndex rix(RB);
    for (int64_t e = int64_t(blockIdx.x) * blockDim.x + threadIdx.x; e < total; e += rix.stride) {
        const int r = rix(e);
        double v = sa * (ca ? ca[r] : 1.0) * a[e];
        if (b) v += sb * (cb ? cb[r] : 1.0) * b[e];
        out[e] = v;
    }
}

// v = inv * sv ; w = v - zfac * w (w = v on the first call) ; Qk = v
__global__ void k_lsqr_vw(const double *sv, const double *inv, const double *zfac, double *v, double *w, double *Qk,
                          int first, int64_t total, int RB) {
    for (int64_t e = int64_t(blockIdx.x) * blockDim.x + threadIdx.x; e < total; e += int64_t(gridDim.x) * blockDim.x) {
        const int r = int(e % RB);
        const double vv = inv[r] * sv[e];
        v[e] = vv;
        w[e] = first ? vv : vv - zfac[r] * w[e];
        if (Qk) Qk[e] = vv;
    }
}

// part[b][j][r] = sum over the rows of block b of Q[j][row][r] s[row][r] for j < k, and
// part[b][k + j][r] the same with the newest basis vector Q[k-1] in place of s: the
// first Gram-Schmidt coefficients and the new row of the Gram matrix in one read of Q.
__global__ void __launch_bounds__(256) k_multidot2_partial(const double *Q, const double *sv, int k, int64_t rows,
                                                           int RB, double *part) {
    __shared__ double red[16 * 256];
    const int G = 256 / RB;
    const int r = threadIdx.x % RB, g = threadIdx.x / RB;
    const int64_t chunk = (rows + gridDim.x - 1) / gridDim.x;
    const int64_t a0 = int64_t(blockIdx.x) * chunk, a1 = a0 + chunk < rows ? a0 + chunk : rows;
    if (a0 >= rows) {  // a block without rows (small meshes)
        for (int e = threadIdx.x; e < 2 * k * RB; e += 256) part[int64_t(blockIdx.x) * 2 * k * RB + e] = 0.0;
        return;
    }
    const int64_t stride = rows * RB;
    const double *w = Q + int64_t(k - 1) * stride;
    for (int j0 = 0; j0 < k; j0 += 8) {
        double acc[8] = {0, 0, 0, 0, 0, 0, 0, 0}, gac[8] = {0, 0, 0, 0, 0, 0, 0, 0};
        for (int64_t row = a0 + g; row < a1; row += G) {
            const int64_t e = row * RB + r;
            const double s = sv[e], q = w[e];
#pragma unroll
            for (int jj = 0; jj < 8; ++jj)
                if (j0 + jj < k) {
                    const double qj = Q[int64_t(j0 + jj) * stride + e];
                    acc[jj] = __builtin_fma(qj, s, acc[jj]);
                    gac[jj] = __builtin_fma(qj, q, gac[jj]);
                }
        }
        // all 16 sums go down the tree together: two barriers per level instead of per sum
#pragma unroll
        for (int jj = 0; jj < 8; ++jj) {
            red[jj * 256 + threadIdx.x] = acc[jj];
            red[(8 + jj) * 256 + threadIdx.x] = gac[jj];
        }
        __syncthreads();
        for (int s = 128; s >= RB; s >>= 1) {
            for (int e = threadIdx.x; e < 16 * s; e += 256) {
                const int v = e / s, t = e & (s - 1);
                red[v * 256 + t] += red[v * 256 + t + s];
            }
            __syncthreads();
        }
        for (int e = threadIdx.x; e < 16 * RB; e += 256) {
            const int v = e / RB, t = e % RB, h = v >> 3, jj = v & 7;
            if (j0 + jj < k) part[(int64_t(blockIdx.x) * 2 * k + h * k + j0 + jj) * RB + t] = red[v * 256 + t];
        }
        __syncthreads();
    }
}

// Second Gram-Schmidt pass from the Gram matrix, one thread per (j, right-hand side).
// cg[j] (j < k) are the first-pass coefficients c1 = Q^T s, cg[k + j] = Q_j . Q_{k-1}.
// Stores that row into gram ([kcap][kcap][RB], symmetric) and writes
//   coef = c1 + c2,  c2 = Q^T (s - Q c1) = c1 - (Q^T Q) c1,
// so that s - Q coef equals two classical Gram-Schmidt passes in exact arithmetic.  The
// new row and column are taken from cg, so no thread waits for another's store (with one
// thread per right-hand side walking k x k entries this took 67 us at k = 15).
__global__ void __launch_bounds__(256) k_gram_coef(double *gram, int kcap, const double *cg, int k, int RB,
                                                   double *coef) {
    const int e = int(blockIdx.x) * 256 + int(threadIdx.x), j = e / RB, r = e % RB;
    if (j >= k) return;
    const double vn = cg[int64_t(k + j) * RB + r];
    gram[(int64_t(k - 1) * kcap + j) * RB + r] = vn;
    gram[(int64_t(j) * kcap + (k - 1)) * RB + r] = vn;
    double gc = 0.0;
    const double *row = gram + int64_t(j) * kcap * RB + r;
    for (int i0 = 0; i0 < k; i0 += 8) {
        double g[8], c[8];
#pragma unroll
        for (int q = 0; q < 8; ++q) {
            const int i = i0 + q < k ? i0 + q : k - 1;
            c[q] = cg[int64_t(i) * RB + r];
            g[q] = j == k - 1 ? cg[int64_t(k + i) * RB + r] : i == k - 1 ? vn : row[int64_t(i) * RB];
        }
#pragma unroll
        for (int q = 0; q < 8; ++q)
            if (i0 + q < k) gc = __builtin_fma(g[q], c[q], gc);
    }
    const double c1 = cg[int64_t(j) * RB + r];
    coef[int64_t(j) * RB + r] = c1 + (c1 - gc);
}

// coef[j][r] = sum_b part[b][j][r]; one workgroup per j
__global__ void __launch_bounds__(256) k_multidot_final(const double *part, int nb, int k, int RB, double *coef) {
    __shared__ double red[256];
    const int j = blockIdx.x;
    const int G = 256 / RB;
    const int r = threadIdx.x % RB, g = threadIdx.x / RB;
    red[threadIdx.x] = strided_sum(part + int64_t(j) * RB + r, g, G, nb, int64_t(k) * RB, 0.0);
    __syncthreads();
    for (int s = 128; s >= RB; s >>= 1) {
        if (threadIdx.x < s) red[threadIdx.x] += red[threadIdx.x + s];
        __syncthreads();
    }
    if (threadIdx.x < RB) coef[int64_t(j) * RB + threadIdx.x] = red[threadIdx.x];
}

// s[row][r] -= coef[j][r] * Q[j][row][r], j = 0..k-1 in order
__global__ void k_project(const double *Q, double *sv, const double *coef, int k, int64_t rows, int RB) {
    const int64_t total = rows * RB;
    const RhsIndex rix(RB);
    for (int64_t e = int64_t(blockIdx.x) * blockDim.x + threadIdx.x; e < total; e += rix.stride) {
        const int r = rix(e);
        double s = sv[e];
        for (int j = 0; j < k; ++j) s -= coef[int64_t(j) * RB + r] * Q[int64_t(j) * total + e];
        sv[e] = s;
    }
}

__global__ void k_stats(const double *x, int64_t S, int64_t N, double *mean, double *std) {
    for (int64_t i = int64_t(blockIdx.x) * blockDim.x + threadIdx.x; i < N; i += int64_t(gridDim.x) * blockDim.x) {
        double m = 0.0;
        for (int64_t s = 0; s < S; ++s) m += x[s * N + i];
        m /= double(S);
        double v = 0.0;
        for (int64_t s = 0; s < S; ++s) {
            const double d = x[s * N + i] - m;
            v = __builtin_fma(d, d, v);
        }
        if (mean) mean[i] = m;
        if (std) std[i] = S > 1 ? sqrt(v / double(S - 1)) : 0.0;
    }
}

// Convergence diagnostics of one sample per thread from its (||r_d||, ||r_p||) history.
__global__ void k_diagnostics(const double *diag, int64_t S, int n_it, double sqrt_nd, double tau, double *data,
                              double *prior, double *ext, int32_t *first) {
    const int64_t k = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
    if (k >= S) return;
    const double *h = diag + k * int64_t(n_it) * 2;
    const double b0 = sqrt(h[0] * h[0] + h[1] * h[1]);
    const double ib = b0 > 0.0 ? 1.0 / b0 : 1.0;
    int32_t hit = -1;
    for (int j = 0; j < n_it; ++j) {
        const double nd = h[2 * j], np = h[2 * j + 1];
        if (data) data[k * n_it + j] = nd / sqrt_nd;
        if (prior) prior[k * n_it + j] = np * ib;
        if (ext) ext[k * n_it + j] = sqrt(nd * nd + np * np) * ib;
        if (hit < 0 && nd <= tau * sqrt_nd) hit = j;
    }
    if (first) first[k] = hit;
}

int grid_for(int64_t total, int per_block = 256, int cap = 65536) {
    int64_t g = (total + per_block - 1) / per_block;
    if (g < 1) g = 1;
    return int(g < cap ? g : cap);
}

template <typename T>
RowOps<T> row_ops(const DevOps &op);
template <>
RowOps<double> row_ops<double>(const DevOps &op) {
    return RowOps<double>{op.ell_col, op.xcol, op.ell_val64, op.xval64, op.bslot64, op.dtm64, op.rspec,
                          op.spec, op.rdir};
}
template <>
RowOps<float> row_ops<float>(const DevOps &op) {
    return RowOps<float>{op.ell_col, op.xcol, op.ell_val32, op.xval32, op.bslot32, op.dtm32, op.rspec,
                          op.spec, op.rdir};
}
template <typename T>
const T *sw_of(const DevOps &op);
template <>
const double *sw_of<double>(const DevOps &op) { return op.sw64; }
template <>
const float *sw_of<float>(const DevOps &op) { return op.sw32; }
template <typename T>
const T *injw_of(const DevOps &op);
template <>
const double *injw_of<double>(const DevOps &op) { return op.injw64; }
template <>
const float *injw_of<float>(const DevOps &op) { return op.injw32; }

// bytes of a step's state (two vectors read, one written) for one RHS block
inline double state_bytes(const DevOps &op, int RB, size_t tsize) { return 3.0 * op.n * RB * double(tsize); }

template <typename T, int RB>
VFwdArgs<T> fwd_args_v(const DevOps &op, const void *S, const void *Sp, void *Sn, bool rows, bool sample, int t,
                       void *y, double yscale, int *blocks) {
    using G = VGeo<T, RB>;
    VFwdArgs<T> a;
    a.o = row_ops<T>(op);
    a.snode = op.snode;
    a.sw = sw_of<T>(op);
    a.S = static_cast<const T *>(S); a.Sp = static_cast<const T *>(Sp); a.Sn = static_cast<T *>(Sn);
    a.y = y; a.yscale = yscale;
    a.n = op.n; a.n_obs = op.n_obs;
    a.n_tiles = rows ? (op.n + G::RPB - 1) / G::RPB : 0;
    a.sample = sample; a.t = t;
    a.dt = T(op.dt);
    a.n_samp = sample ? int((int64_t(op.n_obs) * RB + 255) / 256) : 0;
    a.stream = state_bytes(op, RB, sizeof(T)) > kInfinityCacheBytes;
    *blocks = a.n_tiles + a.n_samp;
    return a;
}

// Launches of at most kFewGroups = 512 workgroups, two waves per SIMD, take the variants with
// everything in flight (174 to 249 registers) and the records by row: the wave with the
// longest chain of round trips is what such a launch takes.  15,625 nodes, per forward /
// transposed step: 1 float32 RHS 2.87 / 3.07 -> 2.58 / 2.86 us, 4 RHS 4.6 / 5.0 -> 4.0 /
// 4.2, 16 RHS 4.0 / 4.5 -> 3.7 / 4.2; 4,913 nodes, 16 RHS 4.9 / 4.9 -> 4.2 / 4.2.  With the
// waves to hide the round trips the registers cost more (64,000 nodes, 16 RHS 7.0 -> 7.8).
static inline bool few_waves(const DevOps &op, int workgroups) { return op.rdir && workgroups <= kFewGroups; }

template <typename T, typename OT, int RB>
void fwd_impl_v(const DevOps &op, const void *S, const void *Sp, void *Sn, bool rows, bool sample, int t, void *y,
                double yscale, hipStream_t s) {
    int grid = 0;
    const VFwdArgs<T> a = fwd_args_v<T, RB>(op, S, Sp, Sn, rows, sample, t, y, yscale, &grid);
    if (grid <= 0) return;
    const dim3 g(grid), b(256);
    if (few_waves(op, grid)) hipLaunchKernelGGL((k_fwd_v<T, OT, RB, Var::Few>), g, b, 0, s, a);
    else if (a.stream) hipLaunchKernelGGL((k_fwd_v<T, OT, RB, Var::Stream>), g, b, 0, s, a);
    else hipLaunchKernelGGL((k_fwd_v<T, OT, RB, Var::Plain>), g, b, 0, s, a);
}

template <typename T, typename OT, int RB>
void fwd_impl_vm(const FwdStep *st, int n, hipStream_t s) {
    Multi<VFwdArgs<T>> mm{};
    for (int m = 0; m < n; ++m)
        mm.a[m] = fwd_args_v<T, RB>(*st[m].op, st[m].S, st[m].Sp, st[m].Sn, st[m].rows, st[m].sample, st[m].t,
                                    st[m].y, st[m].yscale, &mm.tiles[m]);
    mm.n = n;
    double sb = 0.0;
    for (int m = 0; m < n; ++m) sb += state_bytes(*st[m].op, RB, sizeof(T));
    const int grid = multi_grid(mm.tiles, n);
    if (grid <= 0) return;
    const dim3 g(grid), b(256);
    if (sb > kInfinityCacheBytes) hipLaunchKernelGGL((k_fwd_vm<T, OT, RB, Var::Stream>), g, b, 0, s, mm);
    else hipLaunchKernelGGL((k_fwd_vm<T, OT, RB, Var::Plain>), g, b, 0, s, mm);
}

template <typename T, int RB>
VAdjArgs<T> adj_args_v(const DevOps &op, const void *S, const void *Sp, void *Sn, bool last, int tb, const void *yh,
                       double yscale) {
    using G = VGeo<T, RB>;
    VAdjArgs<T> a;
    a.o = row_ops<T>(op);
    a.injs = op.injs;
    a.injw = injw_of<T>(op);
    a.S = static_cast<const T *>(S); a.Sp = static_cast<const T *>(Sp); a.Sn = static_cast<T *>(Sn);
    a.yh = yh; a.yscale = yscale;
    a.n = op.n; a.n_obs = op.n_obs; a.last = last;
    a.tb = tb; a.ta = last ? -1 : tb + 1;
    a.n_tiles = (op.n + G::RPB - 1) / G::RPB;
    a.dt = T(op.dt);
    a.stream = state_bytes(op, RB, sizeof(T)) > kInfinityCacheBytes;
    return a;
}

template <typename T, typename YT, int RB>
void adj_impl_v(const DevOps &op, const void *S, const void *Sp, void *Sn, bool last, int tb, const void *yh,
                double yscale, hipStream_t s) {
    const VAdjArgs<T> a = adj_args_v<T, RB>(op, S, Sp, Sn, last, tb, yh, yscale);
    const dim3 g(a.n_tiles), b(256);
    if (last) hipLaunchKernelGGL((k_adj_v<T, YT, RB, Var::Plain, true>), g, b, 0, s, a);
    else if (few_waves(op, a.n_tiles)) hipLaunchKernelGGL((k_adj_v<T, YT, RB, Var::Few, false>), g, b, 0, s, a);
    else if (a.stream) hipLaunchKernelGGL((k_adj_v<T, YT, RB, Var::Stream, false>), g, b, 0, s, a);
    else hipLaunchKernelGGL((k_adj_v<T, YT, RB, Var::Plain, false>), g, b, 0, s, a);
}

template <typename T, typename YT, int RB>
void adj_impl_vm(const AdjStep *st, int n, hipStream_t s) {
    Multi<VAdjArgs<T>> mm{};
    for (int m = 0; m < n; ++m) {
        mm.a[m] = adj_args_v<T, RB>(*st[m].op, st[m].S, st[m].Sp, st[m].Sn, st[m].last, st[m].tb, st[m].yh,
                                    st[m].yscale);
        mm.tiles[m] = mm.a[m].n_tiles;
    }
    mm.n = n;
    double sb = 0.0;
    for (int m = 0; m < n; ++m) sb += state_bytes(*st[m].op, RB, sizeof(T));
    const int grid = multi_grid(mm.tiles, n);
    if (grid <= 0) return;
    const dim3 g(grid), b(256);
    if (st[0].last) hipLaunchKernelGGL((k_adj_vm<T, YT, RB, Var::Plain, true>), g, b, 0, s, mm);
    else if (sb > kInfinityCacheBytes) hipLaunchKernelGGL((k_adj_vm<T, YT, RB, Var::Stream, false>), g, b, 0, s, mm);
    else hipLaunchKernelGGL((k_adj_vm<T, YT, RB, Var::Plain, false>), g, b, 0, s, mm);
}

template <typename T, typename OT, int RB>
void fwd_impl(const DevOps &op, const void *S, const void *Sp, void *Sn, bool rows, bool sample, int t, void *y,
              double yscale, hipStream_t s) {
    if constexpr (RB * sizeof(T) >= 16) {
        // a row of the RHS block fits one wave (64 lanes x 16 bytes): up to 256 float / 128 double
        if constexpr (RB * sizeof(T) <= 1024) fwd_impl_v<T, OT, RB>(op, S, Sp, Sn, rows, sample, t, y, yscale, s);
    } else {
        using G = Geo<RB>;
        FwdArgs<T> a;
        a.o = row_ops<T>(op);
        a.snode = op.snode;
        a.sw = sw_of<T>(op);
        a.S = static_cast<const T *>(S); a.Sp = static_cast<const T *>(Sp); a.Sn = static_cast<T *>(Sn);
        a.y = y; a.yscale = yscale;
        a.n = op.n; a.n_obs = op.n_obs;
        a.n_tiles = rows ? (op.n + G::RPB - 1) / G::RPB : 0;
        a.sample = sample; a.t = t;
        a.dt = T(op.dt);
        a.n_samp = sample ? int((int64_t(op.n_obs) * RB + 255) / 256) : 0;
        const int grid = a.n_tiles + a.n_samp;
        if (grid <= 0) return;
        if (few_waves(op, grid)) hipLaunchKernelGGL((k_fwd<T, OT, RB, true>), dim3(grid), dim3(256), 0, s, a);
        else hipLaunchKernelGGL((k_fwd<T, OT, RB, false>), dim3(grid), dim3(256), 0, s, a);
    }
}

template <typename T, typename YT, int RB>
AdjArgs<T> adj_args(const DevOps &op, const void *S, const void *Sp, void *Sn, bool last, int ta, int tb,
                    const void *yh, double yscale) {
    using G = Geo<RB * sizeof(T) >= 16 ? 1 : RB>;  // the scalar-lane geometry, used only below 16 bytes per row
    AdjArgs<T> a;
    a.o = row_ops<T>(op);
    a.injptr = op.injptr; a.injs = op.injs;
    a.injw = injw_of<T>(op);
    a.S = static_cast<const T *>(S); a.Sp = static_cast<const T *>(Sp); a.Sn = static_cast<T *>(Sn);
    a.yh = yh; a.yscale = yscale;
    a.n = op.n; a.n_obs = op.n_obs; a.last = last; a.ta = ta; a.tb = tb;
    a.n_tiles = (op.n + G::RPB - 1) / G::RPB;
    a.dt = T(op.dt);
    return a;
}

template <typename T, typename YT, int RB>
void adj_impl(const DevOps &op, const void *S, const void *Sp, void *Sn, bool last, int tb, const void *yh,
              double yscale, hipStream_t s) {
    if constexpr (RB * sizeof(T) >= 16) {
        if constexpr (RB * sizeof(T) <= 1024) adj_impl_v<T, YT, RB>(op, S, Sp, Sn, last, tb, yh, yscale, s);
    } else {
        const AdjArgs<T> a = adj_args<T, YT, RB>(op, S, Sp, Sn, last, last ? -1 : tb + 1, tb, yh, yscale);
        if (few_waves(op, a.n_tiles)) hipLaunchKernelGGL((k_adj<T, YT, RB, true>), dim3(a.n_tiles), dim3(256), 0, s, a);
        else hipLaunchKernelGGL((k_adj<T, YT, RB, false>), dim3(a.n_tiles), dim3(256), 0, s, a);
    }
}

template <typename T, typename YT, int RB>
void adj_init(const DevOps &op, void *q0, void *qm1, const void *yh, double yscale, hipStream_t s) {
    const AdjArgs<T> a = adj_args<T, YT, RB>(op, nullptr, nullptr, nullptr, false, -1, op.n_steps - 1, yh, yscale);
    hipLaunchKernelGGL((k_adj_init<T, YT, RB>), dim3(grid_for(int64_t(op.n) * RB)), dim3(256), 0, s, a,
                       static_cast<T *>(q0), static_cast<T *>(qm1));
}

template <typename T, typename OT, int RB>
void fwd_multi(const FwdStep *st, int n, hipStream_t s) {
    if constexpr (RB * sizeof(T) >= 16 && RB * sizeof(T) <= 1024) fwd_impl_vm<T, OT, RB>(st, n, s);
}
template <typename T, typename YT, int RB>
void adj_multi(const AdjStep *st, int n, hipStream_t s) {
    if constexpr (RB * sizeof(T) >= 16 && RB * sizeof(T) <= 1024) adj_impl_vm<T, YT, RB>(st, n, s);
}

#define PAT_RB_SWITCH(RBV, CALL)               \
    switch (RBV) {                             \
        case 1: { constexpr int RB_ = 1; CALL; break; }   \
        case 2: { constexpr int RB_ = 2; CALL; break; }   \
        case 4: { constexpr int RB_ = 4; CALL; break; }   \
        case 8: { constexpr int RB_ = 8; CALL; break; }   \
        case 16: { constexpr int RB_ = 16; CALL; break; } \
        case 32: { constexpr int RB_ = 32; CALL; break; } \
        case 64: { constexpr int RB_ = 64; CALL; break; } \
        case 128: { constexpr int RB_ = 128; CALL; break; } \
        case 256: { constexpr int RB_ = 256; CALL; break; } \
        default: break;                                   \
    }

}  // namespace

void launch_fwd_step(Prec prec, int RB, const DevOps &op, const void *S, const void *Sp, void *Sn, bool rows,
                     bool sample, int t, void *y, bool y_is_f64, double yscale, hipStream_t s) {
    if (rows && halo_step_supported(prec, RB, op)) {  // the sampling launch that ends a sweep has no rows
        launch_fwd_halo(prec, RB, op, S, Sp, Sn, sample, t, y, y_is_f64, yscale, s);
        return;
    }
    if (prec == Prec::F64) {
        PAT_RB_SWITCH(RB, (fwd_impl<double, double, RB_>(op, S, Sp, Sn, rows, sample, t, y, yscale, s)));
    } else if (y_is_f64) {
        PAT_RB_SWITCH(RB, (fwd_impl<float, double, RB_>(op, S, Sp, Sn, rows, sample, t, y, yscale, s)));
    } else {
        PAT_RB_SWITCH(RB, (fwd_impl<float, float, RB_>(op, S, Sp, Sn, rows, sample, t, y, yscale, s)));
    }
}

void launch_adj_init(Prec prec, int RB, const DevOps &op, void *q0, void *qm1, const void *yhat, bool y_is_f64,
                     double yscale, hipStream_t s) {
    if (prec == Prec::F64) {
        PAT_RB_SWITCH(RB, (adj_init<double, double, RB_>(op, q0, qm1, yhat, yscale, s)));
    } else if (y_is_f64) {
        PAT_RB_SWITCH(RB, (adj_init<float, double, RB_>(op, q0, qm1, yhat, yscale, s)));
    } else {
        PAT_RB_SWITCH(RB, (adj_init<float, float, RB_>(op, q0, qm1, yhat, yscale, s)));
    }
}

void launch_adj_step(Prec prec, int RB, const DevOps &op, const void *S, const void *Sp, void *Sn, bool last, int tb,
                     const void *yhat, bool y_is_f64, double yscale, hipStream_t s) {
    if (halo_step_supported(prec, RB, op)) {
        launch_adj_halo(prec, RB, op, S, Sp, Sn, last, tb, yhat, y_is_f64, yscale, s);
        return;
    }
    if (prec == Prec::F64) {
        PAT_RB_SWITCH(RB, (adj_impl<double, double, RB_>(op, S, Sp, Sn, last, tb, yhat, yscale, s)));
    } else if (y_is_f64) {
        PAT_RB_SWITCH(RB, (adj_impl<float, double, RB_>(op, S, Sp, Sn, last, tb, yhat, yscale, s)));
    } else {
        PAT_RB_SWITCH(RB, (adj_impl<float, float, RB_>(op, S, Sp, Sn, last, tb, yhat, yscale, s)));
    }
}

bool multi_step_supported(Prec prec, int RB) { return RB * (prec == Prec::F64 ? 8 : 4) >= 16; }

int max_rhs_block(Prec prec) { return prec == Prec::F64 ? 128 : 256; }

void launch_fwd_multi(Prec prec, int RB, bool y_is_f64, const FwdStep *st, int n, hipStream_t s) {
    if (prec == Prec::F64) {
        PAT_RB_SWITCH(RB, (fwd_multi<double, double, RB_>(st, n, s)));
    } else if (y_is_f64) {
        PAT_RB_SWITCH(RB, (fwd_multi<float, double, RB_>(st, n, s)));
    } else {
        PAT_RB_SWITCH(RB, (fwd_multi<float, float, RB_>(st, n, s)));
    }
}

void launch_adj_multi(Prec prec, int RB, bool y_is_f64, const AdjStep *st, int n, hipStream_t s) {
    if (prec == Prec::F64) {
        PAT_RB_SWITCH(RB, (adj_multi<double, double, RB_>(st, n, s)));
    } else if (y_is_f64) {
        PAT_RB_SWITCH(RB, (adj_multi<float, double, RB_>(st, n, s)));
    } else {
        PAT_RB_SWITCH(RB, (adj_multi<float, float, RB_>(st, n, s)));
    }
}

void launch_pack(bool in_f64, bool out_f64, const void *in, int64_t R, int64_t rb0, int RB, int64_t cols,
                 const int32_t *perm, void *out, hipStream_t s) {
    const dim3 g(unsigned((cols + 63) / 64)), b(256);
    if (in_f64 && out_f64)
        hipLaunchKernelGGL((k_pack<double, double>), g, b, 0, s, (const double *)in, R, rb0, RB, cols, perm, (double *)out);
    else if (in_f64)
        hipLaunchKernelGGL((k_pack<double, float>), g, b, 0, s, (const double *)in, R, rb0, RB, cols, perm, (float *)out);
    else if (out_f64)
        hipLaunchKernelGGL((k_pack<float, double>), g, b, 0, s, (const float *)in, R, rb0, RB, cols, perm, (double *)out);
    else
        hipLaunchKernelGGL((k_pack<float, float>), g, b, 0, s, (const float *)in, R, rb0, RB, cols, perm, (float *)out);
}

void launch_unpack(bool in_f64, bool out_f64, const void *in, int64_t R, int64_t rb0, int RB, int64_t cols,
                   const int32_t *perm, void *out, hipStream_t s) {
    const dim3 g(unsigned((cols + 63) / 64)), b(256);
    if (in_f64 && out_f64)
        hipLaunchKernelGGL((k_unpack<double, double>), g, b, 0, s, (const double *)in, R, rb0, RB, cols, perm, (double *)out);
    else if (in_f64)
        hipLaunchKernelGGL((k_unpack<double, float>), g, b, 0, s, (const double *)in, R, rb0, RB, cols, perm, (float *)out);
    else if (out_f64)
        hipLaunchKernelGGL((k_unpack<float, double>), g, b, 0, s, (const float *)in, R, rb0, RB, cols, perm, (double *)out);
    else
        hipLaunchKernelGGL((k_unpack<float, float>), g, b, 0, s, (const float *)in, R, rb0, RB, cols, perm, (float *)out);
}

void launch_fill(double *x, int64_t count, double v, hipStream_t s) {
    hipLaunchKernelGGL(k_fill, dim3(grid_for(count)), dim3(256), 0, s, x, count, v);
}

void launch_cast_to_state(Prec prec, const double *x, void *P, int64_t count, hipStream_t s) {
    if (prec == Prec::F64)
        hipLaunchKernelGGL((k_cast<double>), dim3(grid_for(count)), dim3(256), 0, s, x, (double *)P, count);
    else
        hipLaunchKernelGGL((k_cast<float>), dim3(grid_for(count)), dim3(256), 0, s, x, (float *)P, count);
}

void launch_normals(uint64_t seed, int kind, int64_t k0, int64_t S, int64_t len, double *out, hipStream_t s) {
    hipLaunchKernelGGL(k_normals, dim3(grid_for(S * ((len + 3) / 4))), dim3(256), 0, s, seed, kind, k0, S, len, out);
}
void launch_build_rhs_rng(const double *yobs, uint64_t seed, int64_t k0, int64_t S, int64_t rb0, int RB, int64_t M,
                          double isig, double *bd, hipStream_t s) {
    hipLaunchKernelGGL(k_build_rhs_rng, dim3(grid_for(((M + 3) / 4) * RB)), dim3(256), 0, s, yobs, seed, k0, S, rb0, RB,
                       M, isig, bd);
}
void launch_xi_rng(uint64_t seed, int64_t k0, int64_t S, int64_t rb0, int RB, int64_t N, const int32_t *perm,
                   double *xi, hipStream_t s) {
    hipLaunchKernelGGL(k_xi_rng, dim3(grid_for(N * RB)), dim3(256), 0, s, seed, k0, S, rb0, RB, N, perm, xi);
}
void launch_build_rhs(const double *yobs, const double *eta, int64_t S, int64_t rb0, int RB, int64_t M, double isig,
                      double *bd, hipStream_t s) {
    hipLaunchKernelGGL(k_build_rhs, dim3(unsigned((M + 63) / 64)), dim3(256), 0, s, yobs, eta, S, rb0, RB, M, isig, bd);
}

// (the prior kernels take RB a power of two <= 256, as every RHS block is)
void launch_prior(const DevOps &op, int RB, double a, const double *x, double *y, hipStream_t s) {
    hipLaunchKernelGGL(k_prior, dim3(grid_for(int64_t(op.n) * RB)), dim3(256), 0, s, op.rowptr, op.col, op.k1val64,
                       op.sqrtm, op.isqrtm, op.n, RB, a, x, y);
}

void launch_prior_t(const DevOps &op, int RB, double a, const double *x, double *y, hipStream_t s) {
    hipLaunchKernelGGL(k_prior_t, dim3(grid_for(int64_t(op.n) * RB)), dim3(256), 0, s, op.rowptr, op.col, op.k1val64,
                       op.sqrtm, op.isqrtm, op.n, RB, a, x, y);
}

void launch_gext_t_combine(Prec prec, const DevOps &op, int RB, double a, double isig, const void *PH, const double *rp,
                           double *out, hipStream_t s) {
    const dim3 g(grid_for(int64_t(op.n) * RB)), b(256);
    if (prec == Prec::F64)
        hipLaunchKernelGGL((k_gext_t<double>), g, b, 0, s, op.rowptr, op.col, op.k1val64, op.sqrtm, op.isqrtm, op.n, RB,
                           a, isig, (const double *)PH, rp, out);
    else
        hipLaunchKernelGGL((k_gext_t<float>), g, b, 0, s, op.rowptr, op.col, op.k1val64, op.sqrtm, op.isqrtm, op.n, RB,
                           a, isig, (const float *)PH, rp, out);
}

NormParts launch_norms(const double *x, int64_t xrows, const double *y, int64_t yrows, int RB, double *part,
                       hipStream_t s) {
    NormParts n;
    n.na = kDotBlocks;
    n.a = part;
    if (y) {
        n.nb = kDotBlocks;
        n.b = part + int64_t(kDotBlocks) * RB;
    }
    hipLaunchKernelGGL(k_norms, dim3(n.na + n.nb), dim3(256), 0, s, x, xrows, n.na, n.a, y, yrows, n.nb, n.b, RB);
    return n;
}

NormParts launch_diff_sq(const double *a, int lda, int aoff, const double *y, int64_t rows, int RB, double *part,
                         hipStream_t s) {
    NormParts n;
    n.na = kDotBlocks;
    n.a = part;
    hipLaunchKernelGGL(k_diff_sq_partial, dim3(n.na), dim3(256), 0, s, a, lda, aoff, y, rows, RB, part);
    return n;
}

void launch_cols(const double *in, int ldin, int c0, double *out, int64_t rows, int RB, hipStream_t s) {
    hipLaunchKernelGGL(k_cols, dim3(grid_for(rows * RB)), dim3(256), 0, s, in, ldin, c0, out, rows * RB, RB);
}

void launch_norm_store(const NormParts &n, int RB, double *out, hipStream_t s) {
    hipLaunchKernelGGL(k_norm_store, dim3(1), dim3(256), 0, s, n, RB, out);
}

void launch_norm_alpha(const NormParts &n, int RB, const double *gamma, double *alpha, hipStream_t s) {
    hipLaunchKernelGGL(k_norm_alpha, dim3(1), dim3(256), 0, s, n, RB, gamma, alpha);
}

void launch_norm_gamma(const NormParts &n, int RB, double *gamma, double *beta, double *invn, int first,
                       hipStream_t s) {
    hipLaunchKernelGGL(k_norm_gamma, dim3(1), dim3(256), 0, s, n, RB, gamma, beta, invn, first);
}

void launch_norm_resid(const NormParts &n, double *hist, double *diag, int64_t ld, int64_t col, int64_t rb0, int64_t R,
                       int RB, hipStream_t s) {
    hipLaunchKernelGGL(k_norm_resid, dim3(1), dim3(256), 0, s, n, RB, hist, diag, ld, col, rb0, R);
}

void launch_resid(const double *a, const double *b, double *hist, double *diag, int64_t ld, int64_t col, int64_t rb0,
                  int64_t R, int RB, hipStream_t s) {
    hipLaunchKernelGGL(k_resid, dim3(1), dim3(256), 0, s, a, b, hist, diag, ld, col, rb0, R, RB);
}

void launch_lsqr_scalar(LsqrStage st, const LsqrScalars &c, const NormParts &n, int RB, hipStream_t s) {
    hipLaunchKernelGGL(k_lsqr_scalar, dim3(1), dim3(256), 0, s, st, c, n, RB);
}

void launch_lincomb(double *out, const double *a, const double *ca, double sa, const double *b, const double *cb,
                    double sb, int64_t rows, int RB, hipStream_t s) {
    const int64_t total = rows * RB;
    hipLaunchKernelGGL(k_lincomb, dim3(grid_for(total)), dim3(256), 0, s, out, a, ca, sa, b, cb, sb, total, RB);
}

void launch_lsqr_vw(const double *sv, const double *inv, const double *zfac, double *v, double *w, double *Qk,
                    int first, int64_t rows, int RB, hipStream_t s) {
    const int64_t total = rows * RB;
    hipLaunchKernelGGL(k_lsqr_vw, dim3(grid_for(total)), dim3(256), 0, s, sv, inv, zfac, v, w, Qk, first, total, RB);
}

void launch_update_xr(double *x, const double *d, double *rp, const double *qp, const double *alpha, int64_t rows,
                      int RB, hipStream_t s) {
    const int64_t total = rows * RB;
    hipLaunchKernelGGL(k_update_xr, dim3(grid_for(total)), dim3(256), 0, s, x, d, rp, qp, alpha, total, RB);
}

void launch_axpy_neg(double *y, const double *x, const double *alpha, int64_t rows, int RB, hipStream_t s) {
    const int64_t total = rows * RB;
    hipLaunchKernelGGL(k_axpy_neg, dim3(grid_for(total)), dim3(256), 0, s, y, x, alpha, total, RB);
}

void launch_append_dir(const double *sv, double *Qk, double *d, const double *invn, const double *beta, int first,
                       int64_t rows, int RB, hipStream_t s) {
    const int64_t total = rows * RB;
    hipLaunchKernelGGL(k_append, dim3(grid_for(total)), dim3(256), 0, s, sv, Qk, d, invn, beta, first, total, RB);
}

void launch_reorth_coef(const double *Q, const double *sv, int k, int64_t rows, int RB, double *part, double *cg,
                        double *gram, int kcap, double *coef, hipStream_t s) {
    if (k <= 0) return;
    hipLaunchKernelGGL(k_multidot2_partial, dim3(kMultiBlocks), dim3(256), 0, s, Q, sv, k, rows, RB, part);
    hipLaunchKernelGGL(k_multidot_final, dim3(2 * k), dim3(256), 0, s, part, kMultiBlocks, 2 * k, RB, cg);
    hipLaunchKernelGGL(k_gram_coef, dim3((k * RB + 255) / 256), dim3(256), 0, s, gram, kcap, cg, k, RB, coef);
}

void launch_project(const double *Q, double *sv, const double *coef, int k, int64_t rows, int RB, hipStream_t s) {
    if (k <= 0) return;
    hipLaunchKernelGGL(k_project, dim3(grid_for(rows * RB)), dim3(256), 0, s, Q, sv, coef, k, rows, RB);
}

void launch_diagnostics(const double *diag, int64_t S, int n_it, int64_t n_data, double tau, double *data,
                        double *prior, double *ext, int32_t *first, hipStream_t s) {
    hipLaunchKernelGGL(k_diagnostics, dim3(grid_for(S)), dim3(256), 0, s, diag, S, n_it, sqrt(double(n_data)), tau,
                       data, prior, ext, first);
}

void launch_stats(const double *samples, int64_t S, int64_t N, double *mean, double *std, hipStream_t s) {
    hipLaunchKernelGGL(k_stats, dim3(grid_for(N)), dim3(256), 0, s, samples, S, N, mean, std);
}

}  // namespace pat
