// Halo-tile step kernels: blocks whose rows are whole 256-byte chunks (64 to 256
// float32 or 32 to 128 float64 right-hand sides).
//
// The vector-lane kernels gather 16 neighbour rows per row through the CU's texture
// units, which keeps those units busy most of the step.  Here a tile of consecutive
// rows (HaloTiles: at most 32 rows whose distinct neighbour rows, the halo, fit 132
// LDS rows; on the 195,112-node ball 4.7 halo rows per row) copies its halo from
// memory straight into LDS (global_load_lds_dwordx4, 64 lanes x 16 bytes per
// instruction, no registers in between), and every slot reads its neighbour from
// there.  The halo holds rows of the state S (the K part) and, at the rows that its
// boundary slots refer to, rows of the previous state S_prev (the B part).  Each lane
// of a row's 16 holds one slot's operands in registers and hands them to the others by
// DPP row broadcast.  Sums run in the slot order of the vector-lane kernels, with the
// same operations, so both give the same bits.
#include <hip/hip_runtime.h>

#include "pat_internal.h"
#include "pat_kernels.h"
#include "pat_step.h"
#include "pat_tiles.h"

namespace pat {
namespace {

constexpr int kHRows = HaloTiles::kRows;
constexpr int kHMax = HaloTiles::kMax;
constexpr int kHThreads = kHRows * 16;
constexpr int kHWaves = kHThreads / 64;
constexpr int kHPerWave = (kHMax / 4 + kHWaves - 1) / kHWaves;  // halo copy instructions per wave at most
constexpr int kHChunk = 4;  // LDS reads in flight per lane before they are consumed
constexpr uint32_t kNoRow = 0xFFFFFFFFu;
static_assert(kHThreads % 64 == 0 && kHThreads <= 1024, "halo tile geometry");
// Infinity Cache (memory-side last-level cache) of the MI355X
constexpr double kInfinityCacheBytes = 256.0 * 1024 * 1024;

template <typename T>
struct HVec;
template <>
struct HVec<float> {
    using t = float __attribute__((ext_vector_type(4)));
    static constexpr int n = 4;
};
template <>
struct HVec<double> {
    using t = double __attribute__((ext_vector_type(2)));
    static constexpr int n = 2;
};

template <typename T>
struct HaloArgs {
    const int4 *desc;  // per tile: first row, first halo entry, first boundary rank, packed counts
    const int32_t *hrow;
    const uint32_t *meta;  // the tiles' metadata blocks
    const T *eval, *bw, *dtm, *xval, *bslot, *injw, *sw;
    const int32_t *rspec, *xcol, *injs, *snode;
    const int4 *spec;
    const T *S, *Sp;
    T *Sn;
    const void *yh;        // transpose: data
    void *y;               // forward: samples
    double yscale;
    int n_ht, n_obs, sample, t, ta, tb;
    T dt;
};

template <int J>
__device__ __forceinline__ uint32_t row_bcast(uint32_t x) {
    return uint32_t(__builtin_amdgcn_update_dpp(0, int(x), 0x150 + J, 0xF, 0xF, true));
}
template <int J>
__device__ __forceinline__ float row_bcast(float x) { return __uint_as_float(row_bcast<J>(__float_as_uint(x))); }
template <int J>
__device__ __forceinline__ double row_bcast(double x) {
    const unsigned long long b = static_cast<unsigned long long>(__double_as_longlong(x));
    const unsigned long long lo = row_bcast<J>(uint32_t(b)), hi = row_bcast<J>(uint32_t(b >> 32));
    return __longlong_as_double(static_cast<long long>(hi << 32 | lo));
}

template <typename VT, typename T>
__device__ __forceinline__ VT hfma(T w, VT x, VT acc) {
    VT o;
#pragma unroll
    for (int i = 0; i < HVec<T>::n; ++i) o[i] = mad(w, x[i], acc[i]);
    return o;
}

template <bool NT, typename VT>
__device__ __forceinline__ VT load_own(const char *p) {
    if constexpr (NT) return __builtin_nontemporal_load(reinterpret_cast<const VT *>(p));
    else return *reinterpret_cast<const VT *>(p);
}
template <bool NT, typename VT>
__device__ __forceinline__ void store_own(char *p, VT v) {
    if constexpr (NT) __builtin_nontemporal_store(v, reinterpret_cast<VT *>(p));
    else *reinterpret_cast<VT *>(p) = v;
}

__device__ __forceinline__ void lds_copy16(const void *src, void *lds) {
    __builtin_amdgcn_global_load_lds(src, (__attribute__((address_space(3))) void *)lds, 16, 0, 0);
}

// LDS image of one tile: the halo rows (256-byte chunks; K part, then B part) and, in
// float32, its metadata block (HaloTiles) with every row operand, so that the loop
// needs no other load.  The block's float64 values would leave room for one workgroup
// per CU only; there the image holds the boundary rows' B values and local indices, and
// each lane loads its row's operands into registers an item ahead.  (In float32 those
// loads cost more than the block's copies: 36.8 / 38.4 against 35.4 / 36.3 us per
// forward / transposed step of 64 RHS on the 195,112-node ball.)
// A workgroup has two images and two halo row lists, each its own __shared__ variable,
// so that the compiler can tell the copies into one buffer from the reads of the other
// and does not wait for the former before the latter.
template <typename T>
struct HaloBuf;
template <>
struct alignas(16) HaloBuf<float> {
    HVec<float>::t rows[kHMax * 16];
    uint32_t meta[HaloTiles::kMetaBytes / 4];
    __device__ __forceinline__ const float *bw(int nr) const { return reinterpret_cast<const float *>(meta + nr * 24); }
    __device__ __forceinline__ const uint8_t *bloc(int nr, int nbr) const {
        return reinterpret_cast<const uint8_t *>(meta + nr * 24 + nbr * 16);
    }
};
template <>
struct alignas(16) HaloBuf<double> {
    HVec<double>::t rows[kHMax * 16];
    double bws[kHRows * 16];
    uint8_t blocs[kHRows * 16];
    __device__ __forceinline__ const double *bw(int) const { return bws; }
    __device__ __forceinline__ const uint8_t *bloc(int, int) const { return blocs; }
};
struct alignas(16) HaloList {  // copied into 16 bytes per lane
    int32_t r[kHMax];
};
// workgroups per CU that the LDS of two images and two lists allows (160 KiB per CU)
template <typename T>
constexpr int kHPerCU = int(163840 / (2 * (sizeof(HaloBuf<T>) + sizeof(HaloList))));

struct HDesc {
    int r0, nr, h0, nk4, nb4, b0, nbr;
};

// unpack a tile descriptor into wave-uniform values
__device__ __forceinline__ HDesc desc_uniform(const int4 u) {
    const int r0 = __builtin_amdgcn_readfirstlane(u.x), h0 = __builtin_amdgcn_readfirstlane(u.y);
    const int b0 = __builtin_amdgcn_readfirstlane(u.z), f = __builtin_amdgcn_readfirstlane(u.w);
    constexpr int B = HaloTiles::kNrBits, M = (1 << B) - 1;
    return {r0, f & M, h0, (f >> B) & 255, (f >> (B + 8)) & 255, b0, (f >> (B + 16)) & M};
}

// A tile's metadata block (HaloTiles): 96 bytes per row and 80 per boundary row, of all tiles
// before it too.
template <typename T>
__device__ __forceinline__ const char *tile_meta(const HaloArgs<T> &a, const HDesc &d) {
    return reinterpret_cast<const char *>(a.meta) + uint64_t(uint32_t(d.r0) * 6u + uint32_t(d.b0) * 5u) * 16u;
}

// Work items of this workgroup: (chunk c, tile t).  XCD x (workgroups b with
// b % 8 == x) owns the x-th eighth of the tiles, [t_lo, t_lo + ntx), seen as rows
// of G8 consecutive tiles (one per workgroup of the XCD: neighbouring tiles are in
// flight together and share halo rows in its L2).  Two workgroups share a CU, and
// the one dispatched first (k = b / 8 < G8 / 2) runs about a fifth faster than
// the other; so every kRowPeriod-th row goes to the first half only, two tiles
// each, and they take 10 tiles for every 8 of the others.  A workgroup walks its
// tiles in row order, once per 256-byte chunk.
struct HWork {
    int t_lo, ntx, k, G8, per_c, n;
    bool weighted, first_half;
    // local index (tile - t_lo) of this workgroup's j-th tile; increasing in j
    __device__ int local(int j) const { return hwork_local(j, G8, k, weighted, first_half); }
    __device__ HWork(int n_ht, int NC, bool two_per_cu) {
        G8 = int(gridDim.x >> 3);
        const int x = int(blockIdx.x & 7);
        k = int(blockIdx.x >> 3);
        t_lo = int(int64_t(n_ht) * x / 8);
        ntx = int(int64_t(n_ht) * (x + 1) / 8) - t_lo;
        weighted = two_per_cu && G8 % 2 == 0;
        first_half = 2 * k < G8;
        per_c = 0;
        while (local(per_c) < ntx) ++per_c;
        n = per_c * NC;
    }
    __device__ int chunk(int it) const { return it / per_c; }
    __device__ int tile(int it) const { return t_lo + local(it - chunk(it) * per_c); }
};

// Start the copy of a tile's halo row list (nh entries, a multiple of 4 from a
// 16-byte aligned start) into list; one wave issues it.
__device__ __forceinline__ void halo_list_issue(const int32_t *hrow, const HDesc &d, int nh, int32_t *list, int wave,
                                                int lane) {
    if (wave == 1 && 4 * lane < nh) lds_copy16(hrow + d.h0 + 4 * lane, list);
}

// Start the copies of a tile into Lb: its halo rows (row numbers from list; the first
// nk4 from S, the rest from S_prev) at byte offset coff of each row, and the metadata
// block or boundary tables.  Copy instruction h (halo rows 4h .. 4h+3) is issued by
// wave h % 8.
template <typename T, uint32_t RS>
__device__ __forceinline__ void halo_issue(const HaloArgs<T> &a, uint32_t coff, const HDesc &d, const int32_t *list,
                                           HaloBuf<T> &Lb, int wave, int lane) {
    // wave is wave-uniform (callers pass it through readfirstlane), so the tests and
    // the base select below are scalar; the list entries are read in one batch
    int hr[kHPerWave];
#pragma unroll
    for (int m = 0; m < kHPerWave; ++m) {
        const int h = wave + kHWaves * m;
        hr[m] = list[min(4 * h, kHMax - 4) + (lane >> 4)];
    }
    const uint32_t lo = coff + uint32_t(lane & 15) * 16u;
    const int nh = d.nk4 + d.nb4;
#pragma unroll
    for (int m = 0; m < kHPerWave; ++m) {
        const int h = wave + kHWaves * m;
        if (4 * h < nh) {
            const char *base = reinterpret_cast<const char *>(4 * h < d.nk4 ? a.S : a.Sp);
            lds_copy16(base + (uint32_t(hr[m]) * RS + lo), &Lb.rows[h * 64]);
        }
    }
    const int u = kHWaves - 1 - wave;  // 16-byte units, 64 per instruction
    if constexpr (sizeof(T) == 4) {
        const int nu = d.nr * 6 + d.nbr * 5;
        const char *src = tile_meta(a, d) + u * 1024;
        if (u * 64 < nu && u * 64 + lane < nu) lds_copy16(src + uint32_t(lane) * 16u, &Lb.meta[u * 256]);
    } else if (d.nbr) {
        const int nu = d.nbr * 8;
        const char *src = reinterpret_cast<const char *>(a.bw) + uint64_t(uint32_t(d.b0) * 8u + uint32_t(u * 64)) * 16u;
        if (u * 64 < nu && u * 64 + lane < nu) lds_copy16(src + uint32_t(lane) * 16u, &Lb.bws[u * 128]);
        if (wave == 0 && lane < d.nbr) lds_copy16(tile_meta(a, d) + (d.nr * 96 + d.nbr * 64) + uint32_t(lane) * 16u, Lb.blocs);
    }
}

// The operands of one row as held by lane q of its row group: slot q's halo row and K
// value, info word q % 4 and, in float64, dt/m.  Info words: dt/m (float32 bits);
// boundary row of the tile (0xFF: none) | bnum << 8 | overflow entries << 16 | sensor
// weights << 24; first overflow entry; first sensor weight.
template <typename T>
struct HOps {
    uint32_t loc, info;
    T kv, dm;
    // float32: row g of the tile from its metadata block
    __device__ __forceinline__ void from_lds(const HaloBuf<T> &Lb, int nr, int g, int q) {
        loc = reinterpret_cast<const uint8_t *>(Lb.meta + g * 4)[q];
        info = Lb.meta[nr * 4 + g * 4 + (q & 3)];
        kv = reinterpret_cast<const float *>(Lb.meta + nr * 8 + g * 16)[q];
    }
    // float64: row g of tile d from memory (K and dt/m in float64, the rest from the tile's block)
    __device__ __forceinline__ void from_memory(const HaloArgs<T> &a, const HDesc &d, int g, int q) {
        const uint32_t row = uint32_t(d.r0 + g);
        const char *m = tile_meta(a, d);
        loc = *reinterpret_cast<const uint8_t *>(m + uint32_t(g * 16 + q));
        kv = a.eval[int64_t(row) * 16 + 4 * (q & 3) + (q >> 2)];  // slot q of the quad-ordered row
        info = *reinterpret_cast<const uint32_t *>(m + uint32_t((d.nr + g) * 16 + (q & 3) * 4));
        dm = a.dtm[row];
    }
    __device__ __forceinline__ T dtm() const {
        if constexpr (sizeof(T) == 4) return __uint_as_float(row_bcast<0>(info));
        else return dm;
    }
    __device__ __forceinline__ uint32_t word() const { return row_bcast<1>(info); }
    __device__ __forceinline__ int x0() const { return int(row_bcast<2>(info)); }
    __device__ __forceinline__ int inj0() const { return int(row_bcast<3>(info)); }
};

template <typename VT, typename T>
__device__ __forceinline__ VT lds_row(const HaloBuf<T> &Lb, uint32_t off) {
    return *reinterpret_cast<const VT *>(reinterpret_cast<const char *>(Lb.rows) + off);
}

// Pi^T (yhat^{ta} + yhat^{tb}) over the injection entries [e0, e1) of a row, for the
// VEC right-hand sides from rhs0 (yhat^{ta} left out for ta < 0).  All of an entry's data
// are loaded before any are used: with each right-hand side's loads and sum in turn a
// sensor row held its workgroup up (195,112 nodes, 1024 sensors, transposed step: 64
// float32 RHS 35.9 -> 35.5 us, 32 float64 38.2 -> 37.6).
template <typename T, typename YT, int RB, typename VT>
__device__ __forceinline__ VT hinject(const HaloArgs<T> &a, int e0, int e1, int rhs0) {
    VT inj = {};
    const YT *yh = static_cast<const YT *>(a.yh);
    for (int e = e0; e < e1; ++e) {
        const int s = a.injs[e];
        const int64_t sb = (int64_t(a.tb) * a.n_obs + s) * RB + rhs0;
        const int64_t sa = (int64_t(a.ta) * a.n_obs + s) * RB + rhs0;
        const T w = a.injw[e];
        YT yb[HVec<T>::n], ya[HVec<T>::n];
#pragma unroll
        for (int i = 0; i < HVec<T>::n; ++i) yb[i] = yh[sb + i];
        if (a.ta >= 0) {
#pragma unroll
            for (int i = 0; i < HVec<T>::n; ++i) ya[i] = yh[sa + i];
        }
#pragma unroll
        for (int i = 0; i < HVec<T>::n; ++i) {
            T v = static_cast<T>(static_cast<double>(yb[i]) * a.yscale);
            if (a.ta >= 0) v = static_cast<T>(static_cast<double>(ya[i]) * a.yscale) + v;
            inj[i] = mad(w, v, inj[i]);
        }
    }
    return inj;
}

// Pipeline of one workgroup over its work items: fn_list(d, list) starts the copy
// of an item's halo row list, fn_issue(it, d, list, buffer) the copies of its halo,
// fn_pre(it, d) loads its own rows and operands into the "next" registers and
// fn_rot moves them to the "current" ones, fn_compute(it, d, buffer) computes
// item it into registers and fn_store() writes the last computed item.  While
// item it is computed, the copies of item it + 1, the row list of item it + 2 and
// the descriptor of item it + 4 are in flight, and item it - 1's stores drain
// (stores are issued one item late so that their completion is not waited on).
// Even items use (B0, L0), odd items (B1, L1); the loop is unrolled by two so
// that each access names its buffer at compile time.
template <typename Buf, typename List, typename Issue, typename Pre, typename Rot, typename Compute, typename Store>
__device__ __forceinline__ void halo_loop(const HWork &wk, const int4 *D, Buf &B0, Buf &B1, HaloList &L0,
                                          HaloList &L1, List fn_list, Issue fn_issue, Pre fn_pre, Rot fn_rot,
                                          Compute fn_compute, Store fn_store) {
    const int n = wk.n;
    if (n == 0) return;
    auto raw = [&](int it) { return it < n ? D[wk.tile(it)] : int4{0, 0, 0, 0}; };
    HDesc d0 = desc_uniform(raw(0)), d1 = desc_uniform(raw(1)), d2 = desc_uniform(raw(2));
    fn_list(d0, L0.r);
    if (1 < n) fn_list(d1, L1.r);
    __builtin_amdgcn_s_waitcnt(0x0F70);  // vmcnt(0)
    __syncthreads();
    fn_issue(0, d0, L0.r, B0);
    fn_pre(0, d0);
    int4 u3 = raw(3);
    __builtin_amdgcn_s_waitcnt(0x0F70);  // vmcnt(0): the copies of item 0 have landed
    __syncthreads();
    auto step = [&](int it, Buf &Bc, Buf &Bn, HaloList &Lc, HaloList &Ln) {
        fn_rot();
        if (it + 1 < n) fn_issue(it + 1, d1, Ln.r, Bn);
        if (it + 2 < n) fn_list(d2, Lc.r);
        if (it > 0) fn_store();
        if (it + 1 < n) fn_pre(it + 1, d1);
        const int4 u4 = raw(it + 4);
        fn_compute(it, d0, Bc);
        __builtin_amdgcn_s_waitcnt(0x0F70);  // vmcnt(0): the copies of item it + 1 and list it + 2 have landed
        __syncthreads();                     // ... for every wave, and item it's buffer is free
        d0 = d1;
        d1 = d2;
        d2 = desc_uniform(u3);
        u3 = u4;
    };
    for (int it = 0; it < n; it += 2) {
        step(it, B0, B1, L0, L1);
        if (it + 1 < n) step(it + 1, B1, B0, L1, L0);
    }
    fn_store();
}

// One step (FWD: forward; else transposed, with LAST the closing launch: as a run-time
// flag its selects cost 2% of every step).  Each workgroup (512 threads: 32 rows x 16
// lanes of 16 bytes) walks its items through two LDS images.
template <typename T, typename YT, bool FWD, bool LAST, int RB, bool NT>
__global__ void __launch_bounds__(kHThreads) __attribute__((amdgpu_waves_per_eu(4))) k_halo(const HaloArgs<T> a) {
    using VT = typename HVec<T>::t;
    constexpr int V = HVec<T>::n;
    constexpr uint32_t RS = uint32_t(RB * sizeof(T));
    constexpr int NC = int(RS / 256);
    __shared__ HaloBuf<T> B0, B1;
    __shared__ HaloList L0, L1;
    const int tid = int(threadIdx.x), wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63, g = tid >> 4,
              q = tid & 15;
    const uint32_t q16 = uint32_t(q) * 16u;
    const HWork wk(a.n_ht, NC, kHPerCU<T> == 2);
    const char *Sc = reinterpret_cast<const char *>(a.S), *Spc = reinterpret_cast<const char *>(a.Sp);
    VT prev_cur = {}, prev_nxt = {}, out = {};
    HOps<T> o_cur = {}, o_nxt = {};
    uint32_t out_at = kNoRow;  // byte offset of the pending result, kNoRow: none
    auto fn_list = [&](const HDesc &d, int32_t *list) {
        halo_list_issue(a.hrow, d, d.nk4 + d.nb4, list, wave, lane);
    };
    auto fn_issue = [&](int it, const HDesc &d, const int32_t *list, HaloBuf<T> &Bn) {
        halo_issue<T, RS>(a, uint32_t(wk.chunk(it)) * 256u, d, list, Bn, wave, lane);
    };
    auto fn_pre = [&](int it, const HDesc &d) {
        if (g < d.nr) {
            const uint32_t row = uint32_t(d.r0 + g);
            prev_nxt = load_own<NT, VT>(Spc + (row * RS + uint32_t(wk.chunk(it)) * 256u + q16));
            if constexpr (sizeof(T) == 8) o_nxt.from_memory(a, d, g, q);
        }
    };
    auto fn_rot = [&]() {
        prev_cur = prev_nxt;
        if constexpr (sizeof(T) == 8) o_cur = o_nxt;
    };
    auto fn_store = [&]() {
        if (out_at != kNoRow) store_own<NT, VT>(reinterpret_cast<char *>(a.Sn) + out_at, out);
    };
    auto fn_compute = [&](int it, const HDesc &d, const HaloBuf<T> &Lb) {
        out_at = kNoRow;
        if (g >= d.nr) return;
        const uint32_t coff = uint32_t(wk.chunk(it)) * 256u;
        HOps<T> o;
        if constexpr (sizeof(T) == 4) o.from_lds(Lb, d.nr, g, q);
        else o = o_cur;
        const uint32_t koff = o.loc * 256u, hw = o.word();
        const int row = d.r0 + g, nx = int((hw >> 16) & 0xFFu), x0 = o.x0();
        VT acc = {}, bacc = {}, cur;
        static_for<0, 16, kHChunk>([&](auto J0) {
            constexpr int j0 = decltype(J0)::value;
            VT xs[kHChunk];
            static_for<0, kHChunk>([&](auto J) { xs[J.value] = lds_row<VT>(Lb, row_bcast<j0 + J.value>(koff) + q16); });
            if constexpr (j0 == 0) cur = xs[0];
            static_for<0, kHChunk>([&](auto J) { acc = hfma(row_bcast<j0 + J.value>(o.kv), xs[J.value], acc); });
        });
        for (int k = 0; k < nx; k += 4) {  // four entries' loads at a time, clamped to the row's last
            T w[4];
            int cl[4];
            VT xv[4];
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const int e = x0 + min(k + j, nx - 1);
                cl[j] = a.xcol[e];
                w[j] = a.xval[e];
            }
#pragma unroll
            for (int j = 0; j < 4; ++j)
                xv[j] = *reinterpret_cast<const VT *>(Sc + (uint32_t(cl[j]) * RS + coff + q16));
#pragma unroll
            for (int j = 0; j < 4; ++j)
                if (k + j < nx) acc = hfma(w[j], xv[j], acc);
        }
        const int br = int(hw & 0xFFu);
        if (br != 0xFF) {
            int nb = int((hw >> 8) & 0xFFu);
            asm volatile("" : "+v"(nb));  // else the 16 tests below are byte compares, with a register per constant
            uint32_t ko = koff;
            // read the K part's rows again instead of keeping the K sums' reads live
            asm volatile("" : "+v"(ko));
            const uint32_t bo = (uint32_t(d.nk4) + Lb.bloc(d.nr, d.nbr)[br * 16 + q]) * 256u;
            const T bwq = Lb.bw(d.nr)[br * 16 + q];
            // slots j >= nb carry B = 0: the vector-lane kernels add 0 * 0 there, which leaves
            // bacc unchanged (it starts at +0 and a sum that starts at +0 never becomes -0),
            // so skipping them keeps the bits
            static_for<0, 16, kHChunk>([&](auto J0) {
                constexpr int j0 = decltype(J0)::value;
                if (j0 < nb) {
                    VT df[kHChunk];
                    static_for<0, kHChunk>([&](auto J) {
                        if (j0 + J.value < nb) {
                            const VT xv = lds_row<VT>(Lb, row_bcast<j0 + J.value>(ko) + q16);
                            const VT yv = lds_row<VT>(Lb, row_bcast<j0 + J.value>(bo) + q16);
#pragma unroll
                            for (int i = 0; i < V; ++i) df[J.value][i] = bdiff(xv[i], yv[i], LAST);
                        }
                    });
                    static_for<0, kHChunk>([&](auto J) {
                        if (j0 + J.value < nb) bacc = hfma(row_bcast<j0 + J.value>(bwq), df[J.value], bacc);
                    });
                }
            });
            if (nb > 16) {
                const T *bx = a.bslot + a.spec[2 * (a.rspec[row] - 1)].x + 16;
                for (int k = 0; k < nb - 16; ++k) {
                    const uint32_t off = uint32_t(a.xcol[x0 + k]) * RS + coff + q16;
                    const VT xv = *reinterpret_cast<const VT *>(Sc + off), yv = *reinterpret_cast<const VT *>(Spc + off);
                    VT dv;
#pragma unroll
                    for (int i = 0; i < V; ++i) dv[i] = bdiff(xv[i], yv[i], LAST);
                    bacc = hfma(bx[k], dv, bacc);
                }
            }
        }
        VT inj = {};
        if constexpr (!FWD) {
            const int e0 = o.inj0(), e1 = e0 + int(hw >> 24);
            if (e1 > e0) inj = hinject<T, YT, RB, VT>(a, e0, e1, (int(coff) / 16 + q) * V);
        }
        const T dm = o.dtm();
        VT res;
#pragma unroll
        for (int i = 0; i < V; ++i) {
            const T src = T(0.5) * inj[i];
            if constexpr (LAST) res[i] = adj_result(cur[i], prev_cur[i], acc[i], bacc[i], src, dm, a.dt);
            else res[i] = step_update(cur[i], prev_cur[i], acc[i], bacc[i], src, dm, a.dt);
        }
        out = res;
        out_at = uint32_t(row) * RS + coff + q16;
    };
    halo_loop(wk, a.desc, B0, B1, L0, L1, fn_list, fn_issue, fn_pre, fn_rot, fn_compute, fn_store);
    if constexpr (FWD) {
        if (a.sample) {
            // y = Pi (S^n + S^{n-1})/2 of the incoming state, one lane per (sensor, rhs)
            const int64_t total = int64_t(a.n_obs) * RB;
            YT *yo = static_cast<YT *>(a.y);
            for (int64_t e = int64_t(blockIdx.x) * kHThreads + tid; e < total; e += int64_t(gridDim.x) * kHThreads) {
                const int s = int(e / RB), rr = int(e % RB);
                T y = T(0);
                for (int k = 0; k < 4; ++k) {
                    const int64_t id = int64_t(a.snode[4 * s + k]) * RB + rr;
                    y = mad(a.sw[4 * s + k], T(0.5) * (a.S[id] + a.Sp[id]), y);
                }
                yo[(int64_t(a.t) * a.n_obs + s) * RB + rr] = static_cast<YT>(static_cast<double>(y) * a.yscale);
            }
        }
    }
}

template <typename T>
HaloArgs<T> halo_args(const DevOps &op, const void *S, const void *Sp, void *Sn) {
    HaloArgs<T> a{};
    a.desc = op.ht_desc; a.hrow = op.ht_hrow; a.meta = op.ht_meta;
    a.rspec = op.rspec; a.xcol = op.xcol; a.injs = op.injs; a.snode = op.snode; a.spec = op.spec;
    if constexpr (sizeof(T) == 8) {
        a.eval = op.ell_val64; a.bw = op.ht_bw; a.dtm = op.dtm64; a.xval = op.xval64; a.bslot = op.bslot64;
        a.injw = op.injw64; a.sw = op.sw64;
    } else {
        a.eval = op.ell_val32; a.dtm = op.dtm32; a.xval = op.xval32; a.bslot = op.bslot32;
        a.injw = op.injw32; a.sw = op.sw32;
    }
    a.S = static_cast<const T *>(S); a.Sp = static_cast<const T *>(Sp); a.Sn = static_cast<T *>(Sn);
    a.n_ht = op.n_ht; a.n_obs = op.n_obs;
    a.dt = T(op.dt);
    return a;
}

// workgroups of a launch: as many per CU as run together, a multiple of the 8 XCDs
template <typename T>
int halo_grid(const DevOps &op) { return (kHPerCU<T> * op.n_cu + 7) / 8 * 8; }

template <typename T, typename YT, int RB>
void fwd_halo(const DevOps &op, const HaloArgs<T> &a, bool stream, hipStream_t s) {
    const dim3 g(halo_grid<T>(op)), b(kHThreads);
    if (stream) hipLaunchKernelGGL((k_halo<T, YT, true, false, RB, true>), g, b, 0, s, a);
    else hipLaunchKernelGGL((k_halo<T, YT, true, false, RB, false>), g, b, 0, s, a);
}
template <typename T, typename YT, int RB>
void adj_halo(const DevOps &op, const HaloArgs<T> &a, bool last, bool stream, hipStream_t s) {
    const dim3 g(halo_grid<T>(op)), b(kHThreads);
    if (last) hipLaunchKernelGGL((k_halo<T, YT, false, true, RB, false>), g, b, 0, s, a);
    else if (stream) hipLaunchKernelGGL((k_halo<T, YT, false, false, RB, true>), g, b, 0, s, a);
    else hipLaunchKernelGGL((k_halo<T, YT, false, false, RB, false>), g, b, 0, s, a);
}

// calls fn(T{}, RB) for the block widths of whole 256-byte chunks
template <typename F>
void halo_dispatch(Prec prec, int RB, F &&fn) {
    if (prec == Prec::F64) {
        switch (RB) {
            case 32: fn(double{}, std::integral_constant<int, 32>{}); break;
            case 64: fn(double{}, std::integral_constant<int, 64>{}); break;
            case 128: fn(double{}, std::integral_constant<int, 128>{}); break;
            default: break;
        }
    } else {
        switch (RB) {
            case 64: fn(float{}, std::integral_constant<int, 64>{}); break;
            case 128: fn(float{}, std::integral_constant<int, 128>{}); break;
            case 256: fn(float{}, std::integral_constant<int, 256>{}); break;
            default: break;
        }
    }
}

bool beyond_cache(const DevOps &op, Prec prec, int RB) {
    return 3.0 * op.n * RB * (prec == Prec::F64 ? 8 : 4) > kInfinityCacheBytes;
}

}  // namespace

// Rows of one to four 256-byte chunks, and at least 1.5 tiles per workgroup: below that
// the pipelines have nothing to overlap, and the vector-lane kernels win or are even at
// every width, although a wider row gives a workgroup more items.  Halo tiles against
// vector lanes, us per forward / transposed step:
//               4,913 nodes              15,625 (564 tiles)        19,683
//   float32  64   5.2 /  5.5,  4.7 /  5.4    7.0 /  7.0,  7.1 /  7.1    7.6 /  7.8,  7.5 /  7.8
//           128   7.3 /  8.1,  5.8 /  6.5   11.2 / 11.6, 10.5 / 10.6   11.9 / 12.4, 12.0 / 12.4
//           256  11.7 / 13.6,  8.2 /  8.5   19.4 / 20.3, 17.2 / 16.7   20.5 / 21.3, 20.5 / 21.5
//   float64  32   5.5 /  5.4,  4.9 /  5.4    7.4 /  7.0,  7.2 /  7.3    7.7 /  7.8,  7.8 /  7.8
//            64   7.6 /  7.9,  6.1 /  6.6   11.4 / 11.2, 10.6 / 10.6   12.3 / 12.0, 12.2 / 12.1
//           128  12.4 / 12.8,  8.4 /  8.4   19.5 / 20.0, 17.7 / 17.2   20.8 / 21.1, 20.9 / 21.1
// (one chunk on 9,261 to 12,167 nodes, one tile per workgroup: the tiles are ahead, 5.6 / 6.0
// against 5.8 / 6.6 with 64 float32 RHS; wider rows lose on the smaller and are within 4% on
// the larger).  On 29,791 nodes (1,075 tiles) and above the tiles win (15.4 against 17.7
// us, float64, 64 RHS).
bool halo_step_supported(Prec prec, int RB, const DevOps &op) {
    const int row = RB * (prec == Prec::F64 ? 8 : 4);
    return row >= 256 && row <= 1024 && op.n_cu > 0 && op.n_ht >= 3 * op.n_cu;
}

void launch_fwd_halo(Prec prec, int RB, const DevOps &op, const void *S, const void *Sp, void *Sn, bool sample, int t,
                     void *y, bool y_is_f64, double yscale, hipStream_t s) {
    const bool stream = beyond_cache(op, prec, RB);
    halo_dispatch(prec, RB, [&](auto tv, auto rb) {
        using T = decltype(tv);
        HaloArgs<T> a = halo_args<T>(op, S, Sp, Sn);
        a.sample = sample; a.t = t; a.y = y; a.yscale = yscale;
        if constexpr (sizeof(T) == 8) fwd_halo<T, double, rb.value>(op, a, stream, s);
        else if (y_is_f64) fwd_halo<T, double, rb.value>(op, a, stream, s);
        else fwd_halo<T, float, rb.value>(op, a, stream, s);
    });
}

void launch_adj_halo(Prec prec, int RB, const DevOps &op, const void *S, const void *Sp, void *Sn, bool last, int tb,
                     const void *yhat, bool y_is_f64, double yscale, hipStream_t s) {
    const bool stream = beyond_cache(op, prec, RB);
    halo_dispatch(prec, RB, [&](auto tv, auto rb) {
        using T = decltype(tv);
        HaloArgs<T> a = halo_args<T>(op, S, Sp, Sn);
        a.yh = yhat; a.yscale = yscale; a.tb = tb; a.ta = last ? -1 : tb + 1;
        if constexpr (sizeof(T) == 8) adj_halo<T, double, rb.value>(op, a, last, stream, s);
        else if (y_is_f64) adj_halo<T, double, rb.value>(op, a, last, stream, s);
        else adj_halo<T, float, rb.value>(op, a, last, stream, s);
    });
}

}  // namespace pat
