// sph_device.hpp -- gfx950 kernels of the weakly compressible delta-SPH hot path.
//
// Stages of one step (diffSPH, arXiv 2507.21684):
//   assign / scan / scatter / order  cell list by counting sort (App. B, steps 1-2)
//   build_list                       neighbour query over the cell stencil (App. B, step 3)
//   sweep                            Wendland-C4 kernel and gradient (App. A.1), summation
//                                    density, continuity + delta diffusion, Tait pressure and
//                                    artificial viscosity (Sec. 2.3), semi-implicit Euler (Sec. 3.4)
//   adj_prologue / adj_sweep         the vector-Jacobian product of one step (Sec. 2.2) with
//                                    the kernel Hessian (Sec. 3.3)
//
// Every pair sum is a gather: a particle adds its neighbours' terms in the order of its
// neighbour list, which is canonical (stencil cells by relative offset, then particles by
// original index), so results are deterministic and independent of tiling and batching.
// No floating-point atomics are used anywhere.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

namespace sph {

constexpr int kFlagNonfinite = 1;
constexpr int kFlagOverflow = 2;
constexpr int kFlagSkin = 4;  // a particle moved more than its half skin since its list was built

// Half skins of reused lists: particle i may move h_i between two list builds, and a pair is
// listed when r < H + h_i + h_j.  Uniform skins take h_i = hmax (half the simulation's skin);
// speed-scaled skins take h_i = min(hmax, kSkinFloor hmax + kSkinMargin R dt |v_i|) from the
// particle's speed when the lists are built (R the rebuild interval).  A pair that comes
// within H before the next build is therefore listed as long as neither particle has moved more
// than its own h_i, which every step checks (kFlagSkin).  The additive floor is every particle's
// allowance for acceleration over the interval: with hmax sized for 1.3 times the largest speed,
// a particle at rest may accelerate steadily to about a third of that speed; the margin covers
// 30 % more than its own speed.
constexpr double kSkinMargin = 1.3;
constexpr double kSkinFloor = 0.125;

template <typename T> struct Vec4;
template <> struct Vec4<float> { using type = float4; };
template <> struct Vec4<double> { using type = double4; };
template <typename T> using vec4_t = typename Vec4<T>::type;

// Per-simulation constants.  Every floating-point field is rounded once, on the host,
// in the working precision T (H2 = H*H, invL = 1/L computed in T).
template <typename T>
struct SimConst {
    T L, invL, H, H2, invH, cinv;
    T m, rho0, inv_rho0, c0sq, dt;
    T kW;       // C_d / H^d
    T kG;       // C_d / H^(d+2)
    T invW0;    // 1 / W(dx), dx = (m / rho0)^(1/dim) the initial spacing (particle shifting)
    T epsH2;    // eps H^2
    T cA;       // alpha H c0 rho0
    T cD;       // 2 delta H c0
    T Bt;       // rho0 c0^2 / 7
    T HL2;      // (H (1 + skin))^2: list radius squared (= H2 without a skin)
    T hmax;     // skin H / 2: the largest half skin of a particle (the cells are sized for it)
    int64_t p0, n;      // packed particle range
    int32_t cell0;      // first global cell slot
    int32_t blk0;       // first global cell block
    int32_t nc;         // cells per box side
    int32_t sub;        // stencil half-width in cells (cell side >= H / sub)
    int32_t B;          // cells per block side
    int32_t nb;         // blocks per box side
    int32_t Bd;         // B^dim
    int32_t ncu;        // stencil cells per cell, (2 sub + 1)^dim
};

// Stencil entry: global cell id in the low 26 bits, periodic image shift (-1, 0, +1 box
// lengths, stored + 1) in two bits per axis above it.
constexpr int kStencilIdBits = 26;
constexpr int32_t kStencilIdMask = (1 << kStencilIdBits) - 1;

// Stencil cell u (u = 0 .. (2 sub + 1)^dim - 1, offsets in lexicographic order z, y, x) of the
// cell at coordinates cc of simulation S, as a stencil entry.  Cells are numbered block-major:
// blocks of B^dim cells in Morton order (blk_rank maps a row-major block index to its rank),
// cells row-major inside a block.
// Cells per block side: 4 in 2D, 2 in 3D (the host sets SimConst::B to the same values).
template <int DIM>
constexpr int kBlockSide = DIM == 3 ? 2 : 4;

// Offsets (x, y, z) of stencil cell u for a stencil of SW cells per side (SW = 2 sub + 1 = 3 or
// 5, a constant here so that the divisions are multiplications).
template <int DIM, int SW>
__device__ __forceinline__ void stencil_offsets(int u, int sub, int* o)
{
    const unsigned v = (unsigned)u;
    o[0] = (int)(v % SW) - sub;
    o[1] = (int)((v / SW) % SW) - sub;
    o[2] = (DIM == 3) ? (int)(v / (SW * SW)) - sub : 0;
}

template <int DIM, typename T, int EXT = 0>
__device__ __forceinline__ int32_t stencil_entry(const SimConst<T>& S, const int32_t* __restrict__ blk_rank,
                                                 const int* cc, int u)
{
    // EXT = 1: the (SW + 1)^DIM union stencil of a group of 2^DIM cells whose lowest cell is cc
    int o[3];
    if (S.sub == 2) stencil_offsets<DIM, 5 + EXT>(u, 2, o);
    else stencil_offsets<DIM, 3 + EXT>(u, 1, o);
    int c[3] = {0, 0, 0}, sh[3] = {0, 0, 0};
#pragma unroll
    for (int k = 0; k < DIM; ++k) {
        int r = cc[k] + o[k];
        if (r < 0) {
            r += S.nc;
            sh[k] = -1;
        } else if (r >= S.nc) {
            r -= S.nc;
            sh[k] = 1;
        }
        c[k] = r;
    }
    constexpr unsigned B = kBlockSide<DIM>;
    const int bx = (int)((unsigned)c[0] / B), by = (int)((unsigned)c[1] / B), bz = (DIM == 3) ? (int)((unsigned)c[2] / B) : 0;
    const int lin = (DIM == 3) ? (bz * S.nb + by) * S.nb + bx : by * S.nb + bx;
    const int rk = blk_rank[S.blk0 + lin];
    const int wl = (DIM == 3) ? ((c[2] - bz * B) * B + (c[1] - by * B)) * B + (c[0] - bx * B)
                              : (c[1] - by * B) * B + (c[0] - bx * B);
    const int id = S.cell0 + rk * (DIM == 3 ? B * B * B : B * B) + wl;
    return id | ((sh[0] + 1) << kStencilIdBits) | ((sh[1] + 1) << (kStencilIdBits + 2)) |
           ((sh[2] + 1) << (kStencilIdBits + 4));
}

// Simulation index of every particle and every cell slot: the last simulation whose first
// particle (cell slot) is at or before it.  Empty simulations share their first index with the
// next one, so the last such simulation is the one that owns the index.
template <typename T>
__global__ void k_sim_index(int64_t N, int64_t ncell, int32_t nsims, const SimConst<T>* __restrict__ sims,
                            int32_t* __restrict__ psim, int32_t* __restrict__ cell_sim)
{
    const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (t < N) {
        int lo = 0, hi = nsims - 1;
        while (lo < hi) {
            const int mid = (lo + hi + 1) >> 1;
            if (sims[mid].p0 <= t) lo = mid;
            else hi = mid - 1;
        }
        psim[t] = lo;
    }
    if (t < ncell) {
        int lo = 0, hi = nsims - 1;
        while (lo < hi) {
            const int mid = (lo + hi + 1) >> 1;
            if (sims[mid].cell0 <= t) lo = mid;
            else hi = mid - 1;
        }
        cell_sim[t] = lo;
    }
}

template <typename T, int DIM>
struct StatePtrs {
    T* x[3];
    T* v[3];
    T* rho;
};

// ---------------------------------------------------------------- helpers

// Workgroup index remapped so that each XCD (workgroups are dispatched round-robin over
// the 8 XCDs) receives one contiguous range of the logical index space: neighbouring
// tiles then share an L2.
__device__ __forceinline__ int xcd_remap(int wg, int nwg)
{
    const int nx = 8;
    int x = wg % nx, y = wg / nx;
    int q = nwg / nx, r = nwg % nx;
    return x * q + (x < r ? x : r) + y;
}

template <typename T>
__device__ __forceinline__ T wrap_pos(T x, T L, T invL)
{
#pragma clang fp contract(off)
    T k = floor(x * invL);
    T s = L * k;
    return x - s;
}

template <typename T>
__device__ __forceinline__ int cell_coord(T u, T cinv, int nc)
{
    T f = floor(u * cinv);
    int c = (int)f;
    c = c < 0 ? 0 : c;
    c = c > nc - 1 ? nc - 1 : c;
    return c;
}

template <typename T, int DIM>
__device__ __forceinline__ int global_cell(const SimConst<T>& S, const int32_t* __restrict__ blk_rank, int cx, int cy,
                                           int cz)
{
    constexpr int B = kBlockSide<DIM>;
    int bx = (int)((unsigned)cx / B), by = (int)((unsigned)cy / B), bz = (DIM == 3) ? (int)((unsigned)cz / B) : 0;
    int wx = cx - bx * B, wy = cy - by * B, wz = (DIM == 3) ? cz - bz * B : 0;
    int lin = (DIM == 3) ? ((bz * S.nb + by) * S.nb + bx) : (by * S.nb + bx);
    int rank = blk_rank[S.blk0 + lin];
    int w = (DIM == 3) ? ((wz * B + wy) * B + wx) : (wy * B + wx);
    return S.cell0 + rank * (DIM == 3 ? B * B * B : B * B) + w;
}

// r^2 of the minimum-image pair vector, every operation rounded in T (no contraction):
//   d = u_i - u_j; d = d - shift; r2 = ((d0 d0) + d1 d1) + d2 d2
// The shift (0 or +-L per axis) is the periodic image of the stencil cell the candidate
// was found in; for any pair within the support it equals L rint((u_i - u_j) / L).
template <typename T, int DIM>
__device__ __forceinline__ T dist2_exact(const T* ui, const T* uj, const T* sh)
{
#pragma clang fp contract(off)
    T r2 = T(0);
#pragma unroll
    for (int k = 0; k < DIM; ++k) {
        T d = ui[k] - uj[k];
        d = d - sh[k];
        T dd = d * d;
        r2 = r2 + dd;
    }
    return r2;
}

// FP32 sweeps use the hardware reciprocal and square root (about 1 ulp); FP64 keeps IEEE
// division and square root.
template <typename T> __device__ __forceinline__ T fast_rcp(T x) { return T(1) / x; }
template <> __device__ __forceinline__ float fast_rcp<float>(float x) { return __builtin_amdgcn_rcpf(x); }
template <typename T> __device__ __forceinline__ T fast_sqrt(T x) { return sqrt(x); }
template <> __device__ __forceinline__ float fast_sqrt<float>(float x) { return __builtin_amdgcn_sqrtf(x); }

// Volume of a particle from its position record.  The 2D record (u, V, p V) holds it; the 3D
// record (u, rho) holds the density, and V = m / rho is recomputed with the arithmetic of the
// kernel that wrote the record, so it is the value that kernel had.
template <typename T, int DIM>
__device__ __forceinline__ T rec_volume(const vec4_t<T>& a, T m)
{
    return DIM == 3 ? m * fast_rcp(a.w) : a.z;
}

template <typename T>
__device__ __forceinline__ T tait(const SimConst<T>& S, T rho)
{
    T s = rho * S.inv_rho0;
    T s2 = s * s;
    T s3 = s2 * s;
    T s6 = s3 * s3;
    return S.Bt * (s6 * s - T(1));
}

template <typename T>
__device__ __forceinline__ T tait_slope(const SimConst<T>& S, T rho)
{
    T s = rho * S.inv_rho0;
    T s2 = s * s;
    T s3 = s2 * s;
    return S.c0sq * (s3 * s3);
}

// Inclusive scan of 32-bit sums over the wavefront by DPP (row shifts, then the row totals
// broadcast to the rows above): six dependent adds instead of six LDS round trips.
__device__ __forceinline__ int32_t wave_incl_scan(int32_t v)
{
    v += __builtin_amdgcn_update_dpp(0, v, 0x111, 0xF, 0xF, false);   // row_shr:1
    v += __builtin_amdgcn_update_dpp(0, v, 0x112, 0xF, 0xF, false);   // row_shr:2
    v += __builtin_amdgcn_update_dpp(0, v, 0x114, 0xF, 0xF, false);   // row_shr:4
    v += __builtin_amdgcn_update_dpp(0, v, 0x118, 0xF, 0xF, false);   // row_shr:8
    v += __builtin_amdgcn_update_dpp(0, v, 0x142, 0xA, 0xF, false);   // row_bcast:15 into rows 1, 3
    v += __builtin_amdgcn_update_dpp(0, v, 0x143, 0xC, 0xF, false);   // row_bcast:31 into rows 2, 3
    return v;
}

__device__ __forceinline__ int64_t wave_incl_scan(int64_t v)
{
    const int lane = threadIdx.x & 63;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        int64_t t = __shfl_up(v, o, 64);
        if (lane >= o) v += t;
    }
    return v;
}

// The simulation of sorted particle i; a plan of one simulation passes no table (psim null).
__device__ __forceinline__ int sim_of(const int32_t* __restrict__ psim, int64_t i) { return psim ? psim[i] : 0; }

// ---------------------------------------------------------------- fill

template <typename I>
__global__ void k_fill(I* __restrict__ p, int64_t n, I val)
{
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) p[i] = val;
}

// ---------------------------------------------------------------- cell assignment

// The members of the cells, collected while they are counted: cell c keeps the original indices of its
// first arrivals in row c of `rows`, cap places.  Later ones (dense clusters) are chained, in four chains by
// turns, whose heads are the row's last four places, with the links, by position in the source order, in
// `link`; the chains' lengths follow from the cell's count, so neither rows nor links are ever cleared.
// (Four, because a chain is a load after the other: a sort of 10 000 particles with 1000 of them in one cell
// took 153 us with one chain, 115 with four.)  cap is a multiple of 4; or 1, a single chain;
// or 0 where arrivals keep their place in the cell in `link` and are scattered into contiguous `rows` once the
// cell starts are known (k_scatter): for the sort by destination, and in plans of many cells.
struct CellMembers {
    int32_t* rows;
    int32_t* link;
    int32_t cap;
    __device__ __forceinline__ int chains() const { return cap < 4 ? 1 : 4; }
    __device__ __forceinline__ int places() const { return cap - chains(); }   // before the heads
};

__device__ __forceinline__ void add_member(const CellMembers& m, int cell, int slot, int32_t p, int32_t orig)
{
    int32_t* row = m.rows + (int64_t)cell * m.cap;
    if (m.cap == 0) m.link[p] = slot;
    else if (slot < m.places()) row[slot] = orig;
    else m.link[p] = atomicExch(&row[m.places() + (slot & (m.chains() - 1))], p);
}

template <typename T, int DIM>
__global__ __launch_bounds__(256) void k_assign(int64_t N, StatePtrs<T, DIM> st, const int32_t* __restrict__ psim,
                                                const SimConst<T>* __restrict__ sims,
                                                const int32_t* __restrict__ blk_rank, int32_t* __restrict__ cell_count,
                                                int32_t* __restrict__ cell_of, CellMembers members,
                                                const int32_t* __restrict__ orig_in, int32_t* __restrict__ status)
{
    int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (p >= N) return;
    const int s = psim[p];
    const SimConst<T>& S = sims[s];
    int c[3] = {0, 0, 0};
    bool bad = false;
#pragma unroll
    for (int k = 0; k < DIM; ++k) {
        T x = st.x[k][p];
        if (!isfinite(x)) {
            bad = true;
            x = T(0);
        }
        T u = wrap_pos(x, S.L, S.invL);
        c[k] = cell_coord(u, S.cinv, S.nc);
    }
    if (bad) atomicOr(&status[s], kFlagNonfinite);
    int gc = global_cell<T, DIM>(S, blk_rank, c[0], c[1], c[2]);
    cell_of[p] = gc;
    add_member(members, gc, atomicAdd(&cell_count[gc], 1), (int32_t)p, orig_in ? orig_in[p] : (int32_t)p);
}

// ---------------------------------------------------------------- exclusive scan (3 phases)

constexpr int kScanThreads = 256;
constexpr int kScanItems = 8;
constexpr int kScanTile = kScanThreads * kScanItems;

template <typename I>
__device__ __forceinline__ I block_excl_scan(I v, I* smem /* >= 5 */, I* total)
{
    const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
    const I inc = wave_incl_scan(v);
    if (lane == 63) smem[wid] = inc;
    __syncthreads();
    I off = 0, tot = 0;
    const int nw = blockDim.x >> 6;
    for (int w = 0; w < nw; ++w) {
        I t = smem[w];
        if (w < wid) off += t;
        tot += t;
    }
    __syncthreads();
    *total = tot;
    return off + inc - v;
}

// Tile sums, and the workgroup that finishes last (atomic ticket; no waiting on other
// workgroups) turns them into exclusive tile offsets, part[np] = grand total, and resets the
// ticket for the next scan.
template <typename I>
__global__ __launch_bounds__(kScanThreads) void k_scan_reduce_last(const I* __restrict__ in, int64_t n,
                                                                   I* __restrict__ part,
                                                                   unsigned int* __restrict__ ticket)
{
    __shared__ I smem[8];
    __shared__ I carry;
    __shared__ int is_last;
    const int64_t base = (int64_t)blockIdx.x * kScanTile + (int64_t)threadIdx.x * kScanItems;
    I sum = 0;
#pragma unroll
    for (int k = 0; k < kScanItems; ++k)
        if (base + k < n) sum += in[base + k];
    I tot;
    block_excl_scan<I>(sum, smem, &tot);
    if (threadIdx.x == 0) {
        part[blockIdx.x] = tot;
        __threadfence();
        const unsigned int done = atomicAdd(ticket, 1u);
        is_last = (done == gridDim.x - 1) ? 1 : 0;
    }
    __syncthreads();
    if (!is_last) return;
    __threadfence();
    const int64_t np = gridDim.x;
    if (threadIdx.x == 0) carry = 0;
    __syncthreads();
    for (int64_t b = 0; b < np; b += blockDim.x) {
        const int64_t i = b + threadIdx.x;
        const I v = (i < np) ? __atomic_load_n(&part[i], __ATOMIC_RELAXED) : I(0);
        I t2;
        const I ex = block_excl_scan<I>(v, smem, &t2);
        const I c0 = carry;
        if (i < np) part[i] = c0 + ex;
        __syncthreads();
        if (threadIdx.x == 0) carry = c0 + t2;
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        part[np] = carry;
        *ticket = 0u;
    }
}

// out[i] = exclusive prefix of in; out[n] = total; optionally zero `in` afterwards
template <typename I>
__global__ __launch_bounds__(kScanThreads) void k_scan_apply(I* __restrict__ in, int64_t n, const I* __restrict__ part,
                                                             int64_t np, I* __restrict__ out, int zero_in)
{
    __shared__ I smem[8];
    int64_t base = (int64_t)blockIdx.x * kScanTile + (int64_t)threadIdx.x * kScanItems;
    I v[kScanItems];
    I s = 0;
#pragma unroll
    for (int k = 0; k < kScanItems; ++k) {
        v[k] = (base + k < n) ? in[base + k] : I(0);
        s += v[k];
    }
    I tot;
    I ex = block_excl_scan<I>(s, smem, &tot) + part[blockIdx.x];
#pragma unroll
    for (int k = 0; k < kScanItems; ++k) {
        if (base + k < n) {
            out[base + k] = ex;
            if (zero_in) in[base + k] = 0;
        }
        ex += v[k];
    }
    if (blockIdx.x == 0 && threadIdx.x == 0) out[n] = part[np];
}

// ---------------------------------------------------------------- within-cell order and gather

__global__ __launch_bounds__(256) void k_scatter(int64_t N, const int32_t* __restrict__ cell_of,
                                                 const int32_t* __restrict__ cell_start,
                                                 const int32_t* __restrict__ orig_in, CellMembers members)
{
    const int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (p >= N) return;
    members.rows[cell_start[cell_of[p]] + members.link[p]] = orig_in ? orig_in[p] : (int32_t)p;
}

// What a sort writes for a particle besides its state: the original index, the packed records that the
// neighbour sweeps read (wrapped position, volume V = m / rho, p V, velocity), with list reuse the position
// the lists are built from and the half skin, and the place in the source order.
template <typename T>
struct SortedSlot {
    int32_t* orig;
    vec4_t<T>* jd0;
    vec4_t<T>* jd1;
    vec4_t<T>* uref;   // null: no list reuse
    T skin_floor, skin_steps;
    int32_t* before;   // null: not kept
};

// Source particle p, of original index op, put at sorted position d.
template <typename T, int DIM>
__device__ __forceinline__ void put_sorted(int64_t p, int d, int op, const SimConst<T>& S,
                                           const StatePtrs<T, DIM>& src, const StatePtrs<T, DIM>& dst,
                                           const SortedSlot<T>& slot)
{
    T x[3] = {0, 0, 0}, v[3] = {0, 0, 0}, u[3] = {0, 0, 0};
#pragma unroll
    for (int k = 0; k < DIM; ++k) {
        x[k] = src.x[k][p];
        v[k] = src.v[k][p];
        dst.x[k][d] = x[k];
        dst.v[k][d] = v[k];
        u[k] = wrap_pos(isfinite(x[k]) ? x[k] : T(0), S.L, S.invL);
    }
    const T rho = src.rho[p];
    dst.rho[d] = rho;
    slot.orig[d] = op;
    if (slot.before) slot.before[d] = (int32_t)p;
    const T V = S.m * fast_rcp(rho);
    const T pr = tait(S, rho);
    const T pV = pr * V;
    vec4_t<T> a, b;
    if (DIM == 3) {
        a.x = u[0]; a.y = u[1]; a.z = u[2]; a.w = rho;
        b.x = v[0]; b.y = v[1]; b.z = v[2]; b.w = pr;
    } else {
        a.x = u[0]; a.y = u[1]; a.z = V; a.w = pV;
        b.x = v[0]; b.y = v[1]; b.z = rho; b.w = pr;
    }
    slot.jd0[d] = a;
    slot.jd1[d] = b;
    if (slot.uref) {
        // the positions the lists are built from and the particle's half skin (list reuse):
        // speed-scaled with skin_floor = kSkinFloor, skin_steps = kSkinMargin R, uniform (hmax)
        // with skin_floor = 1, skin_steps = 0
        T v2 = T(0);
#pragma unroll
        for (int k = 0; k < DIM; ++k) v2 += v[k] * v[k];
        const T hv = slot.skin_floor * S.hmax + slot.skin_steps * S.dt * sqrt(v2);
        const T h = hv < S.hmax ? hv : S.hmax;   // a non-finite speed keeps hmax
        vec4_t<T> r;
        r.x = u[0]; r.y = u[1]; r.z = u[2]; r.w = h;
        slot.uref[d] = r;
    }
}

// The sort by destination, of a state in the caller's order (original index = place in the source order) whose
// indices k_scatter has put into `rows`: one thread per place there, so that the scattered accesses are
// loads, which the L2 serves (a cell's particles share lines with its neighbours'), and the stores are
// coalesced.  One thread per source particle (k_sort_gather) scatters the stores instead, which costs
// little while the source is the sorted state of the step before, and little in a small plan.  Whole
// sorts by source and by destination, in us: 2D 512^2 34.0 and 30.8, 2D 1000^2 79.4 and 67.3, 2D 1400^2 143
// and 114, 3D 100^3 97 and 83 in lattice order, shuffled 2D 512^2 62.6 and 45.2, 3D 64^3 67.8 and 52.2;
// around the line 2D 290^2 (20 736 cells) 23.8 and 23.6, shuffled 30.1 and 27.0, 3D 56^3 30.1 and
// 29.5, shuffled 50.9 and 40.1.
template <typename T, int DIM>
__global__ __launch_bounds__(256) void k_order_gather(int64_t N, const int32_t* __restrict__ rows,
                                                      const int32_t* __restrict__ cell_of,
                                                      const int32_t* __restrict__ cell_start, StatePtrs<T, DIM> src,
                                                      StatePtrs<T, DIM> dst, SortedSlot<T> slot,
                                                      const int32_t* __restrict__ psim,
                                                      const SimConst<T>* __restrict__ sims)
{
    const int64_t q = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (q >= N) return;
    const int p = rows[q];
    const int c = cell_of[p];
    const int s0 = cell_start[c], s1 = cell_start[c + 1];
    int rank = 0;
#pragma unroll 4
    for (int e = s0; e < s1; ++e) rank += rows[e] < p ? 1 : 0;
    put_sorted<T, DIM>(p, s0 + rank, p, sims[sim_of(psim, q)], src, dst, slot);
}

// Threads of k_sort_gather, and where each of its workgroups scans the counts of all cells by itself: up to
// kSortScanCells cells (their prefixes fit its LDS) and kSortScanReads counts read by all workgroups together.
// There the sort is one launch behind the counting; past either the counts go through the two scan launches
// first.  Sorts behind a step, scanned in the gather and by the launches, us: 2D 320^2 with H = 6 dx
// (11 664 cells, 4.7 M reads) 15.9 against 19.6, 2D 364^2 with H = 6 dx (15 376 cells, 8.0 M reads) 17.9 and 20.2, 3D
// 56^3 with H = 5 dx (7.3 M) 21.0 and 21.1, 2D 450^2 with H = 8 dx (9.9 M) 22.6 and 21.4, 3D 64^3 with H = 6
// dx (10.9 M) 27.1 and 24.0, 2D 1000^2 with H = 16 dx (60 M) 82 and 53.
constexpr int kSortThreads = 256;
constexpr int kSortScanCells = 16384;
constexpr int64_t kSortScanReads = 1 << 23;

// Final sorted position = cell start + rank of the particle's original index among its cell's
// members; moves the state there and packs the per-particle data that the neighbour sweeps read
// (wrapped position, volume V = m / rho, p V, velocity).  One thread per particle in source order.
// With SCAN the cell starts are formed here: a wavefront scans its share of the cells, four per lane and
// turn, into LDS (a prefix per four cells), the workgroup's particles look their cell up there, and the
// workgroups write cell_start between them; the last workgroup to have read the counts clears them for
// the next sort.  Bound: launch and memory latency, a chain of a few dependent loads.  Measured behind
// the counting, before (two scan launches, a scatter of the particle indices, a gather that ranked them
// by three dependent loads each) and now, launch gaps not counted: 2D 101^2 17.3 and 5.5 us, 2D 32^2 FP64
// 13.1 and 4.8, 2D 256^2 19.8 and 10.3, 3D 47^3 25.9 and 13.4, 3D 64^3 (scan launches) 34 and 21.
template <typename T, int DIM, bool SCAN>
__global__ __launch_bounds__(kSortThreads) void k_sort_gather(int64_t N, int32_t ncell, int32_t* __restrict__ cell_count,
                                                      int32_t* __restrict__ cell_start,
                                                      unsigned int* __restrict__ ticket,
                                                      const int32_t* __restrict__ cell_of, CellMembers members,
                                                      const int32_t* __restrict__ orig_in, StatePtrs<T, DIM> src,
                                                      StatePtrs<T, DIM> dst, SortedSlot<T> slot,
                                                      const int32_t* __restrict__ psim,
                                                      const SimConst<T>* __restrict__ sims)
{
    constexpr int kWaves = kSortThreads / 64;
    __shared__ int32_t quads[SCAN ? kSortScanCells / 4 : 1];
    __shared__ int32_t wave_sum[kWaves];
    __shared__ int is_last;
    const int64_t p = (int64_t)blockIdx.x * kSortThreads + threadIdx.x;
    const bool active = p < N;
    const int c = active ? cell_of[p] : 0;
    const int op = !active ? 0 : orig_in ? orig_in[p] : (int)p;
    int s0 = 0, n = 0;
    unsigned int done = 0;
    const int nq = ncell >> 2;   // blocks hold 8 or 16 cells
    if (SCAN) {
        constexpr int U = 8;
        const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
        const int seg = (nq + 64 * kWaves - 1) / (64 * kWaves) * 64;   // quads of a wavefront
        const int4* counts = reinterpret_cast<const int4*>(cell_count);
        const int end = (w + 1) * seg < nq ? (w + 1) * seg : nq;
        int carry = 0;
        for (int q0 = w * seg; q0 < end; q0 += 64 * U) {
            int4 v[U];
#pragma unroll
            for (int k = 0; k < U; ++k) {
                const int q = q0 + 64 * k + lane;
                v[k] = counts[q < end ? q : end - 1];
            }
#pragma unroll
            for (int k = 0; k < U; ++k) {
                const int q = q0 + 64 * k + lane;
                const int sum = q < end ? (v[k].x + v[k].y) + (v[k].z + v[k].w) : 0;
                const int inc = wave_incl_scan(sum);
                if (q < end) quads[q] = carry + inc - sum;
                carry += __builtin_amdgcn_readlane(inc, 63);
            }
        }
        if (lane == 0) wave_sum[w] = carry;
        __syncthreads();
        auto quad_start = [&](int q) {
            int s = quads[q];
#pragma unroll
            for (int k = 0; k + 1 < kWaves; ++k) s += q >= (k + 1) * seg ? wave_sum[k] : 0;
            return s;
        };
        const int4 v = counts[c >> 2];
        s0 = quad_start(c >> 2);
        if ((c & 3) > 0) s0 += v.x;
        if ((c & 3) > 1) s0 += v.y;
        if ((c & 3) > 2) s0 += v.z;
        n = (c & 2) ? ((c & 1) ? +v.w : +v.z) : ((c & 1) ? +v.y : +v.x);
        for (int64_t q = p; q < nq; q += (int64_t)gridDim.x * kSortThreads) {
            const int4 u = counts[q];
            int4 o;
            o.x = quad_start((int)q);
            o.y = o.x + u.x;
            o.z = o.y + u.y;
            o.w = o.z + u.z;
            reinterpret_cast<int4*>(cell_start)[q] = o;
        }
        if (p == 0) cell_start[ncell] = (int32_t)N;
        // every count this workgroup reads has arrived before it takes its ticket
        asm volatile("" : "+v"(n), "+v"(s0));
        __builtin_amdgcn_s_waitcnt(0);
        __syncthreads();
        if (threadIdx.x == 0) done = atomicAdd(ticket, 1u);
    } else if (active) {
        s0 = cell_start[c];
        n = cell_start[c + 1] - s0;
    }
    if (active) {
        int rank = 0;
        if (!SCAN && members.cap == 0) {
            const int32_t* row = members.rows + s0;
#pragma unroll 4
            for (int e = 0; e < n; ++e) rank += row[e] < op ? 1 : 0;
        } else {
            const int32_t* row = members.rows + (int64_t)c * members.cap;
            const int places = members.places(), listed = n < places ? n : places;
            for (int e = 0; e < listed; e += 4) {
                const int4 o = *reinterpret_cast<const int4*>(row + e);
                rank += (o.x < op) + (e + 1 < listed && o.y < op) + (e + 2 < listed && o.z < op) +
                        (e + 3 < listed && o.w < op);
            }
            if (n > listed) {
                const int chains = members.chains();
                int j[4];
#pragma unroll
                for (int q = 0; q < 4; ++q) j[q] = q < chains ? row[places + q] : 0;   // heads past the count: unused
                for (int k = places; k < n; k += chains) {
#pragma unroll
                    for (int q = 0; q < 4; ++q) {
                        if (q < chains && k + q < n) {
                            rank += (orig_in ? orig_in[j[q]] : j[q]) < op ? 1 : 0;
                            if (k + q + chains < n) j[q] = members.link[j[q]];
                        }
                    }
                }
            }
        }
        const int d = s0 + rank;
        put_sorted<T, DIM>(p, d, op, sims[sim_of(psim, p)], src, dst, slot);
    }
    if (SCAN) {
        if (threadIdx.x == 0) is_last = done == gridDim.x - 1;
        __syncthreads();
        if (is_last) {
            for (int q = threadIdx.x; q < nq; q += kSortThreads)
                reinterpret_cast<int4*>(cell_count)[q] = make_int4(0, 0, 0, 0);
            if (threadIdx.x == 0) *ticket = 0u;
        }
    }
}

// A particle's state put at sorted index d of a slot that is already sorted and has lists (a later stage
// of a multistage step, with the lists of the step's first stage): the sorted state and the packed records
// as k_sort_gather writes them, and the displacement since the lists were built checked against its half
// skin.
template <typename T, int DIM>
struct StageSlot {
    const int32_t* orig;
    StatePtrs<T, DIM> state;
    vec4_t<T>* jd0;   // null: the slot holds the stage's state already
    vec4_t<T>* jd1;
    const vec4_t<T>* uref;
};

template <typename T, int DIM>
__device__ __forceinline__ void put_stage(const StageSlot<T, DIM>& slot, int64_t d, const SimConst<T>& S, const T* x,
                                          const T* v, T rho, int32_t* __restrict__ status)
{
    T u[3] = {0, 0, 0};
#pragma unroll
    for (int k = 0; k < DIM; ++k) {
        slot.state.x[k][d] = x[k];
        slot.state.v[k][d] = v[k];
        u[k] = wrap_pos(isfinite(x[k]) ? x[k] : T(0), S.L, S.invL);
    }
    slot.state.rho[d] = rho;
    const T V = S.m * fast_rcp(rho);
    const T pr = tait(S, rho);
    const T pV = pr * V;
    vec4_t<T> a, b;
    if (DIM == 3) {
        a.x = u[0]; a.y = u[1]; a.z = u[2]; a.w = rho;
        b.x = v[0]; b.y = v[1]; b.z = v[2]; b.w = pr;
    } else {
        a.x = u[0]; a.y = u[1]; a.z = V; a.w = pV;
        b.x = v[0]; b.y = v[1]; b.z = rho; b.w = pr;
    }
    slot.jd0[d] = a;
    slot.jd1[d] = b;
    const vec4_t<T> ref = slot.uref[d];
    const T rr[3] = {ref.x, ref.y, ref.z};
    T d2 = T(0);
#pragma unroll
    for (int k = 0; k < DIM; ++k) {
        T dk = u[k] - rr[k];
        dk -= S.L * rint(dk * S.invL);
        d2 += dk * dk;
    }
    if (!(d2 <= ref.w * ref.w)) atomicOr(status, kFlagSkin);
}

// The same for a state in original order.
template <typename T, int DIM>
__global__ __launch_bounds__(256) void k_repack(int64_t N, StatePtrs<T, DIM> src, StageSlot<T, DIM> slot,
                                                const int32_t* __restrict__ psim,
                                                const SimConst<T>* __restrict__ sims, int32_t* __restrict__ status)
{
    int64_t d = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (d >= N) return;
    const int s = sim_of(psim, d);
    const int p = slot.orig[d];
    T x[3] = {0, 0, 0}, v[3] = {0, 0, 0};
#pragma unroll
    for (int k = 0; k < DIM; ++k) {
        x[k] = src.x[k][p];
        v[k] = src.v[k][p];
    }
    put_stage<T, DIM>(slot, d, sims[s], x, v, src.rho[p], &status[s]);
}

template <typename T, int DIM>
__device__ __forceinline__ void unpack_u(const vec4_t<T>& a, T* u)
{
    u[0] = a.x;
    u[1] = a.y;
    if (DIM == 3) u[2] = a.z;
}

// ---------------------------------------------------------------- list rows
//
// A row holds list position k (canonical order) at offset list_offset(k).  Inside every group of 16
// positions the two low and the two high bits of the position change places, so that four consecutive
// offsets hold positions p, p + 4, p + 8, p + 12: with four lanes per particle one 16-byte load is a
// lane's share of the group (positions congruent to the lane modulo 4), and the four lanes still gather
// four consecutive positions at a time, which are mostly consecutive particles of one cell, i.e. one or
// two cache lines.  (Rows in canonical order took a load per entry, or a 4 x 4 transpose by DPP: 18
// vector instructions per lane and group, about a tenth of the pair work.)  The width is a multiple of
// 8; where it is not one of 16, the last 8 positions stay in order.  The build fills a row up to the
// next multiple of 16 positions with the particle itself, whose pair adds exactly zero to every sum,
// so the sweeps test no position against the count.
__device__ __forceinline__ int list_offset(int k, int width)
{
    return k < (width & ~15) ? (k & ~15) | ((k & 3) << 2) | ((k >> 2) & 3) : k;
}

// ---------------------------------------------------------------- neighbour lists

// The pair counter is spread over kPairSlots words, one per 128-byte line, so that the
// wavefronts' integer atomics do not serialise on a single address.
constexpr int kPairSlots = 512;
constexpr int kPairStride = 16;
// Status read without a host wait: the pair total and the status words moved to a staging
// area and cleared, for one copy to the host in stream order.  One workgroup of 256 lanes.
__global__ __launch_bounds__(256) void k_poll_stage(int32_t nsims, int32_t* __restrict__ status,
                                                    unsigned long long* __restrict__ pair_slots,
                                                    unsigned long long* __restrict__ stage_pairs,
                                                    int32_t* __restrict__ stage_status)
{
    __shared__ unsigned long long part[256];
    unsigned long long sum = 0;
    for (int k = threadIdx.x; k < kPairSlots; k += blockDim.x) {
        sum += pair_slots[k * kPairStride];
        pair_slots[k * kPairStride] = 0ull;
    }
    part[threadIdx.x] = sum;
    __syncthreads();
    for (int w = blockDim.x / 2; w > 0; w >>= 1) {
        if ((int)threadIdx.x < w) part[threadIdx.x] += part[threadIdx.x + w];
        __syncthreads();
    }
    if (threadIdx.x == 0) *stage_pairs = part[0];
    for (int k = threadIdx.x; k < nsims; k += blockDim.x) {
        stage_status[k] = status[k];
        status[k] = 0;
    }
}

// Candidates (of the stencil of one cell) whose stencil cell is looked up in a byte table;
// later ones, in dense clusters only, search the prefix sums.
constexpr int kCandTable = 2048;

// One wavefront per cell, or `split` wavefronts that share a cell's particles.  The candidates of the
// cell's particles are the particles of the (2 sub + 1)^dim stencil cells, taken in lexicographic
// order of the cell offset, each cell's particles in sorted order (= original index inside a cell),
// which is the canonical list order.  The candidate stream is cut into tiles of kBuildChunks x 64;
// lane l holds candidates 64 k + l of the tile (k = 0 .. kBuildChunks - 1) in registers (a candidate's
// stencil cell comes from a byte table in LDS, or a search of the prefix sums past it), and the
// wavefront's particles, staged in LDS, are taken one after the other with the same address in
// every lane.  For a particle the tile's chunks are independent tests of 64 candidates each; the
// ballot of the accepted ones gives each its rank, so a chunk appends a contiguous run to the
// particle's row, in candidate order.  Lane p keeps p's running count.  Lists are row-major: list
// position k of particle i is nbr[i * width + list_offset(k, width)].
// Bound: instruction issue (the tests; the matrix cores cannot evaluate the predicate's rounding),
// and in plans of few cells the wavefront's serial chain.  Taking a tile of chunks per particle
// instead of one reads the particle's position and count once per tile and leaves the chunks' tests
// independent of each other: 18 vector and about as many scalar instructions per test of 64
// candidates became 13 and 6.  Measured, one chunk at a time against tiles: 3D 64^3 with skins 267
// and 195 us, 3D 40^3 exact 110 and 75 us, the 512-simulation 2D batch 285 and 229 us (252 with the rows
// transposed and filled up for the sweeps).
// With GROUP (2D) a wavefront serves a group of 2 x 2 cells (cell slots c, c + 1, c + B,
// c + B + 1 of a block, B = 4) over their 6 x 6 (or 4 x 4) union stencil, in the same lexicographic order:
// a particle's own stencil cells are a sub-grid of it in the same relative order, and the extra
// row and column of the union lie at least two cell sides, i.e. at least the list radius, away
// from it, so the strict distance test rejects them (also where a small box repeats a cell in
// the union under another periodic image).  Each particle's list is therefore the one of its own
// cell, while the stencil setup and the candidate stream are shared by four cells.
constexpr int kBuildChunks = 4;

template <typename T, int DIM, bool PERPAIR, bool GROUP>
__global__ __launch_bounds__(64) void k_build_list(const int32_t* __restrict__ cell_sim,
                                                   const int32_t* __restrict__ blk_coord,
                                                   const int32_t* __restrict__ blk_rank,
                                                   const SimConst<T>* __restrict__ sims,
                                                   const int32_t* __restrict__ cell_start,
                                                   const vec4_t<T>* __restrict__ jd0, int32_t width,
                                                   int32_t* __restrict__ nbr, int32_t* __restrict__ nbr_count,
                                                   int32_t* __restrict__ status,
                                                   unsigned long long* __restrict__ pair_counter, int exact,
                                                   const vec4_t<T>* __restrict__ href, int split)
{
    // PERPAIR: lists with per-particle half skins; positions and half skins come from href
    // (written by the sort), and the list radius of a pair is H + h_i + h_j
    const vec4_t<T>* __restrict__ rec = PERPAIR ? href : jd0;
    __shared__ vec4_t<T> pu[65];
    __shared__ int32_t uc_delta[128];   // candidate m of stencil cell u is particle uc_delta[u] + m
    __shared__ int32_t uc_pref[129];
    __shared__ int32_t uc_code[128];
    __shared__ uint8_t uc_of[kCandTable];  // stencil cell of each of the first kCandTable candidates

    constexpr int NC = kBuildChunks;
    constexpr bool kGroup = GROUP && DIM == 2;
    constexpr int kExt = kGroup ? 1 : 0;
    const unsigned wg = (unsigned)xcd_remap(blockIdx.x, gridDim.x);
    const int gw = (int)(wg / (unsigned)split), part = (int)(wg % (unsigned)split);
    // lowest cell slot of the wavefront's cells (2D: group gw & 3 of block gw >> 2)
    const int gc = kGroup ? (gw >> 2) * 16 + ((gw >> 1) & 1) * 8 + (gw & 1) * 2 : gw;
    const int lane = threadIdx.x;
    const int s = cell_sim[gc];
    // particles: the range of cells gc (and gc + 1), then in 2D that of cells gc + 4, gc + 5
    const int i0 = cell_start[gc];
    const int n0 = cell_start[gc + (kGroup ? 2 : 1)] - i0;
    const int i1 = kGroup ? cell_start[gc + 4] : 0;
    const int nall = n0 + (kGroup ? cell_start[gc + 6] - i1 : 0);
    // this wavefront's share of them, [qa, qb)
    const int qa = (int)((int64_t)nall * part / split), qb = (int)((int64_t)nall * (part + 1) / split);
    if (qa == qb) return;
    const SimConst<T>& S = sims[s];
    const T SL = S.L, SH = S.H;
    const int width16 = width & ~15;
    const int sub = S.sub, nc = S.nc;
    const int sw1 = 2 * sub + 1 + kExt;
    const int ncu = kGroup ? sw1 * sw1 : S.ncu;
    const T R2 = exact ? S.H2 : S.HL2;  // list radius: the support, or the support plus the skin
    // the cell's coordinates from its block and its place inside the block
    int cc[3];
    bool inside = true;   // no stencil cell is a periodic image: every shift is zero
    {
        constexpr unsigned B = kBlockSide<DIM>, Bd = DIM == 3 ? B * B * B : B * B;
        const unsigned local = (unsigned)(gc - S.cell0);
        const int rank = (int)(local / Bd);
        const unsigned w = local % Bd;
        const int coord = blk_coord[S.blk0 + rank];
        cc[0] = (coord & 1023) * (int)B + (int)(w % B);
        cc[1] = ((coord >> 10) & 1023) * (int)B + (int)((w / B) % B);
        cc[2] = (DIM == 3) ? ((coord >> 20) & 1023) * (int)B + (int)(w / (B * B)) : 0;
#pragma unroll
        for (int k = 0; k < DIM; ++k) inside = inside && cc[k] >= sub && cc[k] + sub + kExt < nc;
    }

    // stencil cells: particle range and periodic image code, two per lane at most
    int carry = 0;
    const int halves = ncu > 64 ? 2 : 1;
    for (int half = 0; half < halves; ++half) {
        const int u = lane + 64 * half;
        int first = 0, count = 0, code = 0;
        if (u < ncu) {
            code = stencil_entry<DIM, T, kExt>(S, blk_rank, cc, u);
            const int id = code & kStencilIdMask;
            first = cell_start[id];
            count = cell_start[id + 1] - first;
        }
        const int inc = wave_incl_scan(count);
        const int beg = carry + inc - count;
        if (u < 128) {
            uc_delta[u] = first - beg;
            uc_pref[u] = beg;
            uc_code[u] = code;
        }
        const int end = (beg + count < kCandTable) ? beg + count : kCandTable;
        for (int m = beg; m < end; ++m) uc_of[m] = uint8_t(u);
        carry += __builtin_amdgcn_readlane(inc, 63);
    }
    const int M = __builtin_amdgcn_readfirstlane(carry);
    if (lane == 0) uc_pref[ncu] = M;
    __syncthreads();

    // the stencil cell holding candidate m: the last one whose prefix is <= m
    auto cell_of_candidate = [&](int m) {
        if (m < kCandTable) return (int)uc_of[m];
        int lo = 0, hi = ncu - 1;
        while (lo < hi) {
            const int mid = (lo + hi + 1) >> 1;
            if (uc_pref[mid] <= m) lo = mid;
            else hi = mid - 1;
        }
        return lo;
    };

    // sorted index of the unit's particle q (the two ranges in order)
    auto pidx = [&](int q) { return q < n0 ? i0 + q : i1 + (q - n0); };
    int pairs_acc = 0;
    for (int pb = qa; pb < qb; pb += 64) {
        const int nb = __builtin_amdgcn_readfirstlane((qb - pb < 64) ? qb - pb : 64);
        // batch positions [0, split0) are in the first range, [split0, nb) in the second
        const int split0 = __builtin_amdgcn_readfirstlane(n0 - pb < 0 ? 0 : (n0 - pb < nb ? n0 - pb : nb));
        __syncthreads();
        if (lane < nb) pu[lane] = rec[pidx(pb + lane)];
        __syncthreads();
        int cnt = 0;  // lane p: entries of the batch's particle p so far
        for (int c0 = 0; c0 < M; c0 += 64 * NC) {
            int jc[NC], code[NC];
            T uj[NC][3], Aj[NC];
            // Candidates past the stream are put out of every particle's reach (the squared distance
            // overflows).  In 3D, where a wavefront goes through several tiles for few particles, the
            // chunks' lookups and loads go side by side, with the last candidate in place of those past
            // the stream (3D 40^3 75.1 and 70.6 us, 3D 64^3 195 and 189); in 2D that takes 10 registers more
            // and gains nothing (2D 151^2 9.5 and 9.7).
            if (DIM == 3) {
                int m[NC];
#pragma unroll
                for (int k = 0; k < NC; ++k) m[k] = c0 + 64 * k + lane < M ? c0 + 64 * k + lane : M - 1;
                if (M <= kCandTable) {
#pragma unroll
                    for (int k = 0; k < NC; ++k) code[k] = uc_of[m[k]];
                } else {
#pragma unroll
                    for (int k = 0; k < NC; ++k) code[k] = cell_of_candidate(m[k]);
                }
                vec4_t<T> un[NC];
#pragma unroll
                for (int k = 0; k < NC; ++k) jc[k] = uc_delta[code[k]] + m[k];
#pragma unroll
                for (int k = 0; k < NC; ++k) un[k] = rec[jc[k]];
                if (!inside) {
#pragma unroll
                    for (int k = 0; k < NC; ++k) code[k] = uc_code[code[k]];
                }
#pragma unroll
                for (int k = 0; k < NC; ++k) {
                    unpack_u<T, DIM>(un[k], uj[k]);
                    if (c0 + 64 * k + lane >= M) uj[k][0] = T(1e38);
                    Aj[k] = SH + un[k].w;   // PERPAIR: H + h_j
                }
            } else {
#pragma unroll
                for (int k = 0; k < NC; ++k) {
                    vec4_t<T> un;
                    un.x = un.y = un.z = T(1e38);
                    un.w = T(0);
                    jc[k] = 0;
                    code[k] = (1 | (1 << 2) | (1 << 4)) << kStencilIdBits;
                    const int m = c0 + 64 * k + lane;
                    if (m < M) {
                        const int u = cell_of_candidate(m);
                        jc[k] = uc_delta[u] + m;
                        code[k] = uc_code[u];
                        un = rec[jc[k]];
                    }
                    uj[k][2] = T(0);
                    unpack_u<T, DIM>(un, uj[k]);
                    Aj[k] = SH + un.w;
                }
            }
            auto shift_of = [&](int k, int d) {
                return T(((code[k] >> (kStencilIdBits + 2 * d)) & 3) - 1) * SL;
            };
            if (PERPAIR && !inside) {
                // PERPAIR lists only need to hold a superset of the pairs within H (the sweeps test
                // those exactly), so their distance takes the candidate's image once per tile and
                // contracted products; exact lists keep the predicate's own arithmetic
#pragma unroll
                for (int k = 0; k < NC; ++k)
#pragma unroll
                    for (int d = 0; d < DIM; ++d) uj[k][d] = uj[k][d] + shift_of(k, d);
            }
            // The batch positions [p0, p1), whose rows follow each other from row, against the tile's
            // first NA chunks.  Straight-line code for a run that fits the row: the scalar unit issues
            // as many instructions per test as the vector unit, so every branch here counts.
            auto rounds = [&](auto images, auto chunks, int p0, int p1, int32_t* row) {
                constexpr int NA = decltype(chunks)::value;
                vec4_t<T> rn = pu[p0];
                for (int p = p0; p < p1; ++p, row += width) {
                    const vec4_t<T> rp = rn;
                    rn = pu[p + 1];
                    T ui[3] = {T(0), T(0), T(0)};
                    unpack_u<T, DIM>(rp, ui);
                    unsigned long long mask[NA];
                    bool in[NA];
#pragma unroll
                    for (int k = 0; k < NA; ++k) {
                        if (PERPAIR) {
                            const T Rp = Aj[k] + rp.w;
                            const T d0 = ui[0] - uj[k][0];
                            T r2 = d0 * d0;
#pragma unroll
                            for (int d = 1; d < DIM; ++d) {
                                const T dd = ui[d] - uj[k][d];
                                r2 = fma(dd, dd, r2);
                            }
                            in[k] = r2 < Rp * Rp;
                        } else if (decltype(images)::value) {
                            const T sh[3] = {shift_of(k, 0), shift_of(k, 1), shift_of(k, 2)};
                            in[k] = dist2_exact<T, DIM>(ui, uj[k], sh) < R2;
                        } else {
                            const T sh[3] = {T(0), T(0), T(0)};   // d - 0 is d
                            in[k] = dist2_exact<T, DIM>(ui, uj[k], sh) < R2;
                        }
                        mask[k] = __ballot(in[k]);
                    }
                    const int base = __builtin_amdgcn_readlane(cnt, p);
                    int c[NA], total = base;
#pragma unroll
                    for (int k = 0; k < NA; ++k) {
                        c[k] = __popcll(mask[k]);
                        total += c[k];
                    }
                    // an accepted lane's place: after the accepted lanes below it and the earlier chunks
                    int first = base;
                    if (total <= width16) {   // wave-uniform: the whole run fits the row's full groups
#pragma unroll
                        for (int k = 0; k < NA; ++k) {
                            const unsigned pos = __builtin_amdgcn_mbcnt_hi(
                                unsigned(mask[k] >> 32),
                                __builtin_amdgcn_mbcnt_lo(unsigned(mask[k]), unsigned(first)));
                            // 4 list_offset(pos, width), as two bit-field inserts
                            const unsigned mid = ((pos << 4) & 48u) | (pos & ~48u);
                            const unsigned off = (mid & 60u) | ((pos << 2) & ~60u);
                            if (in[k]) *reinterpret_cast<int32_t*>(reinterpret_cast<char*>(row) + off) = jc[k];
                            first += c[k];
                        }
                    } else {
#pragma unroll
                        for (int k = 0; k < NA; ++k) {
                            const unsigned pos = __builtin_amdgcn_mbcnt_hi(
                                unsigned(mask[k] >> 32),
                                __builtin_amdgcn_mbcnt_lo(unsigned(mask[k]), unsigned(first)));
                            if (in[k] && pos < unsigned(width)) row[list_offset((int)pos, width)] = jc[k];
                            first += c[k];
                        }
                    }
                    cnt = (lane == p) ? total : cnt;   // lane p keeps p's count
                }
            };
            auto tile = [&](auto images, auto chunks) {
                rounds(images, chunks, 0, split0, nbr + (int64_t)(i0 + pb) * width);
                if (kGroup) rounds(images, chunks, split0, nb, nbr + (int64_t)pidx(pb + split0) * width);
            };
            auto sized = [&](auto images) {
                const int left = M - c0;   // wave-uniform
                if (left > 192) tile(images, std::integral_constant<int, 4>{});
                else if (left > 128) tile(images, std::integral_constant<int, 3>{});
                else if (left > 64) tile(images, std::integral_constant<int, 2>{});
                else tile(images, std::integral_constant<int, 1>{});
            };
            static_assert(NC == 4, "a tile has four chunks");
            if (PERPAIR || inside) sized(std::false_type{});
            else sized(std::true_type{});
        }
        // each row filled up to a whole group of 16 positions with the particle itself: 16 lanes a row
        for (int p0 = 0; p0 < nb; p0 += 4) {
            const int p = p0 + (lane >> 4), i = pidx(pb + p);
            const int have = __shfl(cnt, p & 63, 64);
            const int pos = have + (lane & 15);
            if (p < nb && pos < ((have + 15) & ~15) && pos < width)
                nbr[(int64_t)i * width + list_offset(pos, width)] = i;
        }
        if (lane < nb) {
            const int i = pidx(pb + lane);
            nbr_count[i] = cnt;
            if (cnt > width) atomicOr(&status[s], kFlagOverflow);
            pairs_acc += cnt - 1;
        }
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) pairs_acc += __shfl_xor(pairs_acc, o, 64);
    if (lane == 0 && pair_counter)
        atomicAdd(&pair_counter[(gc & (kPairSlots - 1)) * kPairStride], (unsigned long long)pairs_acc);
}

// ---------------------------------------------------------------- canonical pair sums
//
// A particle's neighbour sum is split into eight partial sums s_q over list positions
// k = q (mod 8), each accumulated in increasing k, and combined by the balanced tree
// ((s0 + s1) + (s2 + s3)) + ((s4 + s5) + (s6 + s7)).  LPP lanes share a particle
// (LPP in {2, 4, 8}): lane r holds the 8 / LPP partial sums with q = r (mod LPP).  The
// first log2(LPP) levels of the tree combine lanes (xor shuffles; every lane of the group ends
// with the same value because floating-point addition commutes), the remaining levels combine
// a lane's own partial sums.  The result is bitwise the same for every LPP.
constexpr int kLeaves = 8;

template <int LPP, typename T>
__device__ __forceinline__ T combine_leaves(T* a /* [kLeaves / LPP] */)
{
    constexpr int NQ = kLeaves / LPP;
#pragma unroll
    for (int o = 1; o < LPP; o <<= 1) {
#pragma unroll
        for (int q = 0; q < NQ; ++q) a[q] = a[q] + __shfl_xor(a[q], o, 64);
    }
    if (NQ == 1) return a[0];
    if (NQ == 2) return a[0] + a[1];
    return (a[0] + a[1]) + (a[2] + a[3]);
}

// The same for NV sums at once, level by level, so that their shuffles are in flight together (one sum after
// the other waits for each of its own).
template <int LPP, int NV, typename T>
__device__ __forceinline__ void combine_leaves(T (&a)[NV][kLeaves / LPP], T (&out)[NV])
{
    constexpr int NQ = kLeaves / LPP;
#pragma unroll
    for (int o = 1; o < LPP; o <<= 1) {
        T b[NV][NQ];
#pragma unroll
        for (int v = 0; v < NV; ++v)
#pragma unroll
            for (int q = 0; q < NQ; ++q) b[v][q] = __shfl_xor(a[v][q], o, 64);
#pragma unroll
        for (int v = 0; v < NV; ++v)
#pragma unroll
            for (int q = 0; q < NQ; ++q) a[v][q] = a[v][q] + b[v][q];
    }
#pragma unroll
    for (int v = 0; v < NV; ++v)
        out[v] = NQ == 1 ? a[v][0] : NQ == 2 ? a[v][0] + a[v][1 % NQ]
                                             : (a[v][0] + a[v][1 % NQ]) + (a[v][2 % NQ] + a[v][3 % NQ]);
}

// ---------------------------------------------------------------- gathers and fast arithmetic

// Element `idx` of an array whose byte size fits 32 bits: a 32-bit byte offset from the
// array base, so the load uses a scalar base plus a vector offset.
template <typename V>
__device__ __forceinline__ V ldo(const V* __restrict__ base, uint32_t idx)
{
    return *reinterpret_cast<const V*>(reinterpret_cast<const char*>(base) + idx * (uint32_t)sizeof(V));
}

// ---------------------------------------------------------------- traversal of a list row

// One lane's list entries of a group of 16 positions: with 4 lanes a = positions r, r + 4, r + 8,
// r + 12; with 8 lanes the same of r mod 4 (half of it is the lane's); with 2 lanes also b, those
// of r + 2.
struct ListGroup {
    int4 a, b;
};

template <int LPP>
__device__ __forceinline__ ListGroup load_group(const int32_t* __restrict__ row, int g, int r)
{
    ListGroup c;
    const int32_t* p = row + 16 * g;
    c.a = *reinterpret_cast<const int4*>(p + 4 * (r & 3));
    c.b = LPP == 2 ? *reinterpret_cast<const int4*>(p + 4 * (r + 2)) : c.a;
    return c;
}

// Entry u (0 or 1) of the lane's half step e in a group: its list positions r + LPP (2 e + u).
// (The selections are of values: a conditional of lvalues becomes an indexed array in LDS.)
template <int LPP>
__device__ __forceinline__ int group_entry(const ListGroup& c, int e, int u, int r)
{
    const int x = c.a.x, y = c.a.y, z = c.a.z, w = c.a.w;
    if (LPP == 8) {
        const bool odd = (r & 4) != 0;
        return u ? (odd ? +w : +z) : (odd ? +y : +x);
    }
    if (LPP == 4) return e ? (u ? w : z) : (u ? y : x);
    if (u) return e == 0 ? c.b.x : e == 1 ? c.b.y : e == 2 ? c.b.z : c.b.w;
    return e == 0 ? x : e == 1 ? y : e == 2 ? z : w;
}

// Keeps the loads of a record where they were issued: without it the compiler sinks them past the
// exit test that follows, to their first use, and every pair waits for its own gather.
template <int N = 4, typename V>
__device__ __forceinline__ void pin(V& v)
{
    if (N == 4) asm volatile("" : "+v"(v.x), "+v"(v.y), "+v"(v.z), "+v"(v.w));
    else asm volatile("" : "+v"(v.x), "+v"(v.y), "+v"(v.z));
}

// The pairs of lane r of the LPP lanes that share a particle, over the n positions of its row, four at
// a time: gather(j, rec) loads the records of neighbour j, pair(q, rec) adds its terms to the lane's
// partial sum q.  Position k = r + LPP m belongs to partial sum m mod (8 / LPP), in increasing m.
// The four neighbours' records are gathered together, with the next list entries behind them, and
// computed without a branch in between: the more gathers in flight the better where gathers bound the
// sweep (FP32: with two pairs at a time, the next two gathered meanwhile, the 512-simulation batch took
// 375 us a forward sweep against 335).  This part covers the full groups of 16 positions of the row;
// list_tail the last half group.
template <int LPP, typename REC, typename GATHER, typename PAIR>
__device__ __forceinline__ void sweep_burst(const int32_t* __restrict__ row, int width, int n, int r, int self,
                                           GATHER&& gather, PAIR&& pair)
{
    const int groups = width >> 4;
    n = n < 16 * groups ? n : 16 * groups;
    if (n <= 0) return;
    if (LPP == 2) {
        // a group is two turns of 8 positions
        ListGroup c = load_group<LPP>(row, 0, r);
        for (int g = 0;; ++g) {
            const ListGroup nx = load_group<LPP>(row, g + 1 < groups ? g + 1 : g, r);
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                REC rec[4];
                gather(group_entry<LPP>(c, 2 * h, 0, r), rec[0]);
                gather(group_entry<LPP>(c, 2 * h, 1, r), rec[1]);
                gather(group_entry<LPP>(c, 2 * h + 1, 0, r), rec[2]);
                gather(group_entry<LPP>(c, 2 * h + 1, 1, r), rec[3]);
#pragma unroll
                for (int u = 0; u < 4; ++u) pair(u, rec[u]);
                if (16 * g + 8 * (h + 1) >= n) return;
            }
            c = nx;
        }
    } else {
        constexpr int GI = LPP == 8 ? 2 : 1;   // groups per turn
        ListGroup c0 = load_group<LPP>(row, 0, r);
        ListGroup c1 = load_group<LPP>(row, GI == 2 && groups > 1 ? 1 : 0, r);
        for (int g = 0;; g += GI) {
            REC rec[4];
            gather(group_entry<LPP>(c0, 0, 0, r), rec[0]);
            gather(group_entry<LPP>(c0, 0, 1, r), rec[1]);
            if (LPP == 8) {
                // past the row's filled groups the entries are not list entries
                const bool more = 16 * (g + 1) < n;
                gather(more ? group_entry<LPP>(c1, 0, 0, r) : self, rec[2]);
                gather(more ? group_entry<LPP>(c1, 0, 1, r) : self, rec[3]);
            } else {
                gather(group_entry<LPP>(c0, 1, 0, r), rec[2]);
                gather(group_entry<LPP>(c0, 1, 1, r), rec[3]);
            }
            c0 = load_group<LPP>(row, g + GI < groups ? g + GI : 0, r);
            if (GI == 2) c1 = load_group<LPP>(row, g + GI + 1 < groups ? g + GI + 1 : 0, r);
#pragma unroll
            for (int u = 0; u < 4; ++u) pair(LPP == 4 ? u & 1 : 0, rec[u]);
            if (16 * (g + GI) >= n) return;
        }
    }
}

// Whether sweep_piped keeps the next gathers ahead of the pair terms.  Left to itself the compiler lets them
// sink among the terms in some copies of the loop (3D 16^3 FP64, four lanes, right-hand side: 35.6 us a sweep,
// 33.2 with them held; 3D 30^3 60.7 and 56.7).
template <typename REC>
constexpr bool kGatherFirst = true;

// The same pairs two at a time, the records of the next two gathered while these are computed, the
// list entries two groups ahead: for FP64, whose pair terms take several times as long as FP32's, so
// that a wavefront hides its own gathers (2D 32^2, 64 wavefronts: 13.5 us a sweep with four at a time,
// 8.8 with two ahead; 3D 20^3 27.3 and 20.9).
template <int LPP, typename REC, typename GATHER, typename PAIR>
__device__ __forceinline__ void sweep_piped(const int32_t* __restrict__ row, int width, int n, int r, int self,
                                           GATHER&& gather, PAIR&& pair)
{
    constexpr int HS = 8 / LPP;           // half steps of a group
    constexpr int UN = HS == 1 ? 2 : 1;   // groups per turn (an even number of half steps)
    const int groups = width >> 4;
    n = n < 16 * groups ? n : 16 * groups;
    if (n <= 0) return;
    ListGroup c = load_group<LPP>(row, 0, r);
    ListGroup nx = load_group<LPP>(row, groups > 1 ? 1 : 0, r);
    REC rec[2][2];
    gather(group_entry<LPP>(c, 0, 0, r), rec[0][0]);
    gather(group_entry<LPP>(c, 0, 1, r), rec[0][1]);
    for (int g0 = 0;; g0 += UN) {
#pragma unroll
        for (int s = 0; s < HS * UN; ++s) {
            const int g = g0 + s / HS, e = s % HS;
            const bool last = e + 1 == HS;
            int j0, j1;
            if (!last) {
                j0 = group_entry<LPP>(c, e + 1, 0, r);
                j1 = group_entry<LPP>(c, e + 1, 1, r);
            } else {
                // past the row's filled groups the entries are not list entries
                const bool more = 16 * (g + 1) < n;
                j0 = more ? group_entry<LPP>(nx, 0, 0, r) : self;
                j1 = more ? group_entry<LPP>(nx, 0, 1, r) : self;
            }
            gather(j0, rec[(s + 1) & 1][0]);
            gather(j1, rec[(s + 1) & 1][1]);
            if (kGatherFirst<REC>) __builtin_amdgcn_sched_barrier(0);
            if (last) {
                c = nx;
                nx = load_group<LPP>(row, g + 2 < groups ? g + 2 : 0, r);
            }
            pair(LPP == 2 ? (2 * e) % 4 : 0, rec[s & 1][0]);
            pair(LPP == 2 ? (2 * e + 1) % 4 : LPP == 4 ? 1 : 0, rec[s & 1][1]);
            rec[(s + 1) & 1][0].keep();
            rec[(s + 1) & 1][1].keep();
            if (16 * g + 2 * LPP * (e + 1) >= n) return;
        }
    }
}

template <bool PIPED, int LPP, typename REC, typename GATHER, typename PAIR>
__device__ __forceinline__ void sweep_list(const int32_t* __restrict__ row, int width, int n, int r, int self,
                                           GATHER&& gather, PAIR&& pair)
{
    if (PIPED) sweep_piped<LPP, REC>(row, width, n, r, self, gather, pair);
    else sweep_burst<LPP, REC>(row, width, n, r, self, gather, pair);
}

// The last 8 positions (in order) of a row whose width is 8 modulo 16, for the rare particle that
// has so many neighbours.
template <int LPP, typename REC, typename GATHER, typename PAIR>
__device__ __forceinline__ void list_tail(const int32_t* __restrict__ row, int width, int n, int r, int self,
                                          GATHER&& gather, PAIR&& pair)
{
    const int first = width & ~15;
    if (n <= first) return;
#pragma unroll
    for (int m = 0; m < 8 / LPP; ++m) {
        const int k = first + r + LPP * m;
        REC rec;
        gather(k < n ? row[k] : self, rec);
        pair(m, rec);
    }
}

// A neighbour past the support (lists with a skin) has t = 0 and so adds zero without a test, but only
// while its records are finite: 0 times an infinity is NaN.  A particle whose sums come out non-finite
// therefore forms them again from the pairs within the support alone, one at a time and in the same order, so
// that nothing outside the support reaches it.  (A test of the finished sums is a few instructions per
// particle: the sweeps of the 512-simulation batch took 366 and 481 us without it and 367 and 480 with it,
// those of 2D 101^2 6.5 and 8.4 against 6.5 and 8.1.)
template <int LPP, typename REC, typename GATHER, typename PAIR>
__device__ __forceinline__ void walk_again(const int32_t* __restrict__ row, int width, int n, int r, GATHER&& gather,
                                           PAIR&& pair)
{
    n = n < width ? n : width;
    for (int k0 = r; k0 < n; k0 += 8) {
#pragma unroll
        for (int m = 0; m < 8 / LPP; ++m) {
            const int k = k0 + LPP * m;
            if (k < n) {
                REC rec;
                gather(row[list_offset(k, width)], rec);
                pair(m, rec);
            }
        }
    }
}

// Whether a simulation's lists hold pairs past the support.
template <typename T>
__device__ __forceinline__ bool past_support(const SimConst<T>& S) { return S.HL2 > S.H2; }

// An index as a value the compiler knows nothing of.  A pass that forms a particle's sums again loads
// everything anew through one: with the first walk's values kept for it, the walk itself ran out of
// registers (2D adjoint of the 512-simulation batch: 503 us a launch against 481).
template <typename I>
__device__ __forceinline__ I opaque(I v)
{
    asm volatile("" : "+v"(v));
    return v;
}

// Positions the lanes of a particle visit for a row of n entries.
template <typename T, int LPP>
__device__ __forceinline__ int positions_visited(int n, int width)
{
    constexpr int kTurn = (sizeof(T) == 8 ? 2 : 4) * LPP;   // positions of one turn
    const int first = width & ~15, m = n < first ? n : first;
    return (m + kTurn - 1) / kTurn * kTurn + (n > first ? 8 : 0);
}

// Per-simulation constants the pair loops use, held in registers.
template <typename T>
struct PairConst {
    T L, invL, H, invH, epsH2, cA, cD, H2, m;
    T kGF;  // kG (-56/3): grad W = kGF t^5 (1 + 5 q) x_ij = kGF t^5 (6 - 5 t) x_ij
    T hc;   // -30 / H^2 (the Hessian's 560 C_d / H^(d+4) over kGF): it is kGF (t^5 (6 - 5 t) I + hc t^4 x x^T)
};

// Squared distance of a listed pair with the arithmetic of the neighbour predicate (per
// component the minimum image, then the sum of squares in component order, no contraction),
// so that a list with a skin can be filtered to exactly the pairs with r^2 < H^2.
// The minimum-image pair vector is returned in d.
template <typename T, int DIM>
__device__ __forceinline__ T r2_exact(const T* ui, const vec4_t<T>& a, T L, T invL, T* d)
{
#pragma clang fp contract(off)
    const T uj[3] = {a.x, a.y, a.z};
    T r2 = T(0);
#pragma unroll
    for (int k = 0; k < DIM; ++k) {
        T dk = ui[k] - uj[k];
        // L rint(.) is 0 or +-L exactly, so the fused form rounds once, as the separate
        // product and difference do
        dk = fma(-L, rint(dk * invL), dk);
        d[k] = dk;
        T dd = dk * dk;
        r2 = r2 + dd;
    }
    return r2;
}

// The pair vector and its square without the periodic image, with the same roundings: equal to
// r2_exact for every pair within the support of a particle that lies more than the support inside the
// box (the image term is zero there); any other pair comes out at its distance across the box, which is
// past the support too.
template <typename T, int DIM>
__device__ __forceinline__ T r2_inner(const T* ui, const vec4_t<T>& a, T* d)
{
#pragma clang fp contract(off)
    const T uj[3] = {a.x, a.y, a.z};
    T r2 = T(0);
#pragma unroll
    for (int k = 0; k < DIM; ++k) {
        const T dk = ui[k] - uj[k];
        d[k] = dk;
        const T dd = dk * dk;
        r2 = r2 + dd;
    }
    return r2;
}

template <typename T, int DIM, bool IMAGE>
__device__ __forceinline__ T pair_vector(const T* ui, const vec4_t<T>& a, T L, T invL, T* d)
{
    if (IMAGE) return r2_exact<T, DIM>(ui, a, L, invL, d);
    return r2_inner<T, DIM>(ui, a, d);
}

// Whether every lane's particle lies more than the support (and a margin for rounding) inside the box.
template <typename T, int DIM>
__device__ __forceinline__ bool wave_inside(const T* ui, T H, T L)
{
    const T lo = H * T(1.001), hi = L - lo;
    bool in = true;
#pragma unroll
    for (int k = 0; k < DIM; ++k) in = in && ui[k] > lo && ui[k] < hi;
    return __all(in) != 0;
}

// x where it is positive, else zero; x <= 1 (FP32: the clamp of the instruction that makes x).
template <typename T>
__device__ __forceinline__ T positive_part(T x) { return x > T(0) ? x : T(0); }
template <>
__device__ __forceinline__ float positive_part<float>(float x) { return __builtin_amdgcn_fmed3f(x, 0.0f, 1.0f); }

// t = 1 - r / H, zero from the support on: every pair term carries a power of t, so a listed pair past
// the support (lists with a skin) whose records are finite adds exactly zero without a test.
template <typename T>
__device__ __forceinline__ T kernel_t(T r2, T invH)
{
    return positive_part(fma(-invH, fast_sqrt(r2), T(1)));
}

// What the sweep that finishes a step does for the next step when that step reuses the lists
// (null jd0: the next step sorts and rebuilds): the next state goes straight into the next
// tape slot in the same particle order, with its packed records and original indices, and each
// particle's displacement since the list build is checked against its half skin.
template <typename T>
struct NextSlot {
    vec4_t<T>* jd0;
    vec4_t<T>* jd1;
    int32_t* orig;
    const vec4_t<T>* uref;
};

template <typename T>
__device__ __forceinline__ PairConst<T> pair_const(const SimConst<T>& S);

// The constants of simulation s: by scalar loads where the wavefront holds one simulation (vector
// loads of one address still cost the vector L1 an access per four lanes).
template <typename T>
__device__ __forceinline__ PairConst<T> pair_const_of(const SimConst<T>* __restrict__ sims, int s)
{
    const int s0 = __builtin_amdgcn_readfirstlane(s);
    if (__all(s == s0)) return pair_const(sims[s0]);
    return pair_const(sims[s]);
}

template <typename T>
__device__ __forceinline__ PairConst<T> pair_const(const SimConst<T>& S)
{
    PairConst<T> c;
    c.L = S.L;
    c.invL = S.invL;
    c.H = S.H;
    c.invH = S.invH;
    c.epsH2 = S.epsH2;
    c.cA = S.cA;
    c.cD = S.cD;
    c.H2 = S.H2;
    c.m = S.m;
    c.kGF = S.kG * T(-56.0 / 3.0);
    c.hc = T(-30) * (S.invH * S.invH);
    return c;
}

// ---------------------------------------------------------------- forward sweep

// Largest workgroup of the forward and adjoint sweeps.  In FP32 3D with eight lanes 512, i.e. 64 particles, whose
// neighbourhoods overlap in the vector L1 (3D 64^3: 213 and 317 us against 229 and 326 with 256; with
// four lanes, where 256 lanes are 64 particles, 512 is no faster, and neither is it in 2D).
template <typename T, int DIM, int LPP>
constexpr int kSweepThreads = sizeof(T) == 4 && DIM == 3 && LPP == 8 ? 512 : 256;

constexpr int kModeStep = 0;  // integrate into dst (sorted order)
constexpr int kModeRhs = 1;   // write drho, a, rho_sum to caller arrays (original order)

// Weight of a neighbour in the pair sums: its volume in 2D (in its record), 1 / rho in 3D, where
// the sums are multiplied by the particle mass at the end instead.
template <typename T, int DIM>
__device__ __forceinline__ T pair_weight(const vec4_t<T>& a)
{
    return DIM == 3 ? fast_rcp(a.w) : a.z;
}

// ---------------------------------------------------------------- renormalised density gradient
//
// The corrected gradient of App. A.5 applied to the density:
//   G_i = L_i g_i,  L_i = M_i^-1,  M_i = sum_j V_j (x_j - x_i) (x) grad_i W_ij,
//   g_i = sum_j V_j (rho_j - rho_i) grad_i W_ij.
// With grad_i W_ij = gF d (d = x_i - x_j) every pair adds -V_j gF d d^T to M_i (symmetric)
// and V_j gF (rho_j - rho_i) d to g_i.  Same list traversal and eight canonical partial sums
// as the sweeps; a singular M_i gives G_i = 0.  G (and the symmetric L when requested) are
// written in sorted order: 2D L = (L00, L01, L11, 0); 3D L in two records
// (L00, L01, L02, L11), (L12, L22, 0, 0).

template <typename T, int DIM>
struct RenormAcc {
    T M[6];   // 2D: M00, M01, M11; 3D: M00, M01, M02, M11, M12, M22
    T g[3];
};

template <typename T, int DIM>
struct RenormNbr {
    vec4_t<T> a, b;
    __device__ __forceinline__ void keep()
    {
        pin<DIM == 3 ? 4 : 3>(a);
        if (DIM == 2) pin<3>(b);
    }
};

template <typename T, int DIM>
__device__ __forceinline__ bool inv_sym(const T* M, T* L)
{
    if (DIM == 2) {
        const T det = M[0] * M[2] - M[1] * M[1];
        if (!(det != T(0)) || !isfinite(det)) return false;
        const T id = T(1) / det;
        L[0] = M[2] * id;
        L[1] = -M[1] * id;
        L[2] = M[0] * id;
        return true;
    }
    const T a = M[0], b = M[1], c = M[2], d = M[3], e = M[4], f = M[5];
    const T c00 = d * f - e * e, c01 = c * e - b * f, c02 = b * e - c * d;
    const T det = a * c00 + b * c01 + c * c02;
    if (!(det != T(0)) || !isfinite(det)) return false;
    const T id = T(1) / det;
    L[0] = c00 * id;
    L[1] = c01 * id;
    L[2] = c02 * id;
    L[3] = (a * f - c * c) * id;
    L[4] = (b * c - a * e) * id;
    L[5] = (a * d - b * b) * id;
    return true;
}

// y = L x for the symmetric L stored as above.
template <typename T, int DIM>
__device__ __forceinline__ void sym_mul(const T* L, const T* x, T* y)
{
    if (DIM == 2) {
        y[0] = L[0] * x[0] + L[1] * x[1];
        y[1] = L[1] * x[0] + L[2] * x[1];
        y[2] = T(0);
    } else {
        y[0] = L[0] * x[0] + L[1] * x[1] + L[2] * x[2];
        y[1] = L[1] * x[0] + L[3] * x[1] + L[4] * x[2];
        y[2] = L[2] * x[0] + L[4] * x[1] + L[5] * x[2];
    }
}

template <typename T, int DIM, int LPP>
__global__ __launch_bounds__(256) void k_renorm(int64_t N, int32_t width, const int32_t* __restrict__ nbr,
                                                const int32_t* __restrict__ nbr_count,
                                                const vec4_t<T>* __restrict__ jd0, const vec4_t<T>* __restrict__ jd1,
                                                const T* __restrict__ rho3, const int32_t* __restrict__ psim,
                                                const SimConst<T>* __restrict__ sims,
                                                vec4_t<T>* __restrict__ G_out, vec4_t<T>* __restrict__ L_out)
{
    constexpr int NQ = kLeaves / LPP;
    constexpr int NM = DIM == 2 ? 3 : 6;
    const int64_t t = (int64_t)xcd_remap(blockIdx.x, gridDim.x) * blockDim.x + threadIdx.x;
    const int64_t i = t / LPP;
    const int r = (int)(t - i * LPP);
    if (i >= N) return;
    const SimConst<T>& S = sims[psim[i]];
    const PairConst<T> c = pair_const(S);
    T ui[3] = {0, 0, 0};
    unpack_u<T, DIM>(jd0[i], ui);
    const T rhoi = (DIM == 3) ? rho3[i] : jd1[i].z;
    int n = nbr_count[i];
    n = n < width ? n : width;
    const int32_t* row = nbr + i * (int64_t)width;
    RenormAcc<T, DIM> acc[NQ];
    auto gather = [&](int j, RenormNbr<T, DIM>& nb) {
        nb.a = ldo(jd0, (uint32_t)j);
        if (DIM == 2) nb.b = ldo(jd1, (uint32_t)j);
    };
    auto clear = [&]() {
#pragma unroll
        for (int q = 0; q < NQ; ++q) {
#pragma unroll
            for (int a = 0; a < 6; ++a) acc[q].M[a] = T(0);
            acc[q].g[0] = acc[q].g[1] = acc[q].g[2] = T(0);
        }
    };
    auto add = [&](T rho, T invH, const RenormNbr<T, DIM>& nb, const T* d, T r2, RenormAcc<T, DIM>& A) {
        const T tt = kernel_t(r2, invH);
        const T t2 = tt * tt;
        const T rj = (DIM == 3) ? nb.a.w : nb.b.z;
        const T f = pair_weight<T, DIM>(nb.a) * (t2 * t2) * (tt * fma(T(-5), tt, T(6)));
        T fd[3];
#pragma unroll
        for (int k = 0; k < DIM; ++k) fd[k] = f * d[k];
        if (DIM == 2) {
            A.M[0] = fma(-fd[0], d[0], A.M[0]);
            A.M[1] = fma(-fd[0], d[1], A.M[1]);
            A.M[2] = fma(-fd[1], d[1], A.M[2]);
        } else {
            A.M[0] = fma(-fd[0], d[0], A.M[0]);
            A.M[1] = fma(-fd[0], d[1], A.M[1]);
            A.M[2] = fma(-fd[0], d[2], A.M[2]);
            A.M[3] = fma(-fd[1], d[1], A.M[3]);
            A.M[4] = fma(-fd[1], d[2], A.M[4]);
            A.M[5] = fma(-fd[2], d[2], A.M[5]);
        }
        const T dr = rj - rho;
#pragma unroll
        for (int k = 0; k < DIM; ++k) A.g[k] = fma(dr, fd[k], A.g[k]);
    };
    auto pairs = [&](auto image, auto walk) {
        walk([&](int q, RenormNbr<T, DIM>& nb) {
            T d[3] = {0, 0, 0};
            const T r2 = pair_vector<T, DIM, decltype(image)::value>(ui, nb.a, c.L, c.invL, d);
            add(rhoi, c.invH, nb, d, r2, acc[q]);
        });
    };
    auto groups = [&](auto&& pair) { sweep_list<(sizeof(T) == 8), LPP, RenormNbr<T, DIM>>(row, width, n, r, (int)i, gather, pair); };
    auto tail = [&](auto&& pair) { list_tail<LPP, RenormNbr<T, DIM>>(row, width, n, r, (int)i, gather, pair); };
    const T scale = (DIM == 3) ? c.kGF * S.m : c.kGF;
    T M[6], g[3] = {0, 0, 0}, tmp[NQ];
    auto combine = [&]() -> T {
        T sum = T(0);
#pragma unroll
        for (int e = 0; e < NM; ++e) {
#pragma unroll
            for (int q = 0; q < NQ; ++q) tmp[q] = acc[q].M[e];
            M[e] = combine_leaves<LPP>(tmp);
            sum += fabs(M[e]);
        }
#pragma unroll
        for (int k = 0; k < DIM; ++k) {
#pragma unroll
            for (int q = 0; q < NQ; ++q) tmp[q] = acc[q].g[k];
            g[k] = combine_leaves<LPP>(tmp);
            sum += fabs(g[k]);
        }
        return sum;
    };
    clear();
    if (wave_inside<T, DIM>(ui, S.H, S.L)) pairs(std::false_type{}, groups);
    else pairs(std::true_type{}, groups);
    pairs(std::true_type{}, tail);
    if (__builtin_expect(!isfinite(combine()), 0) && past_support(sims[psim[opaque(i)]])) {
        const int64_t i2 = opaque(i);
        const SimConst<T>& S2 = sims[psim[i2]];
        const T invH2 = S2.invH, rho2 = (DIM == 3) ? rho3[i2] : jd1[i2].z;
        T u2[3] = {0, 0, 0};
        unpack_u<T, DIM>(jd0[i2], u2);
        clear();
        walk_again<LPP, RenormNbr<T, DIM>>(
            nbr + i2 * width, width, nbr_count[i2], r, gather, [&](int q, RenormNbr<T, DIM>& nb) {
                T d[3] = {0, 0, 0};
                const T r2 = r2_exact<T, DIM>(u2, nb.a, S2.L, S2.invL, d);
                if (r2 < S2.H2) add(rho2, invH2, nb, d, r2, acc[q]);
            });
        combine();
    }
    if (r != 0) return;
#pragma unroll
    for (int e = 0; e < NM; ++e) M[e] = scale * M[e];
#pragma unroll
    for (int k = 0; k < DIM; ++k) g[k] = scale * g[k];
    T L[6] = {0, 0, 0, 0, 0, 0}, G[3] = {0, 0, 0};
    if (inv_sym<T, DIM>(M, L)) sym_mul<T, DIM>(L, g, G);
    vec4_t<T> o;
    o.x = G[0];
    o.y = G[1];
    o.z = G[2];
    o.w = T(0);
    G_out[i] = o;
    if (L_out) {
        vec4_t<T> l0, l1;
        if (DIM == 2) {
            l0.x = L[0]; l0.y = L[1]; l0.z = L[2]; l0.w = T(0);
            L_out[i] = l0;
        } else {
            l0.x = L[0]; l0.y = L[1]; l0.z = L[2]; l0.w = L[3];
            l1.x = L[4]; l1.y = L[5]; l1.z = T(0); l1.w = T(0);
            L_out[2 * i] = l0;
            L_out[2 * i + 1] = l1;
        }
    }
}

template <typename T, int DIM>
struct FwdAcc {
    T ax[3];
    T rdv, rdd, rs, rdg;
};

// Per-particle sweep record of a neighbour (jd0, jd1; G with the renormalised diffusion).
template <typename T, int DIM, bool RENORM>
struct FwdNbr {
    vec4_t<T> a, b, G;
    int j;
    __device__ __forceinline__ void keep()
    {
        pin(a);
        if (DIM == 3) pin(b);
        else pin<3>(b);
        if (RENORM) pin<3>(G);
    }
};

template <typename T>
struct FwdSelf {
    T u[3], v[3];
    T rho, p;
    T G[3];   // renormalised density gradient
};

// Forward pair terms of (i, j), added to acc:
//   a_i    += ((alpha H c0 rho0 pi_ij - p_i) V_j - p_j V_j) gW
//   drho_i += V_j (v_i - v_j).gW     (times rho_i later)   and   V_j (rho_i - rho_j) x_ij.gW / (r^2 + eps H^2)
//   rho_i  += W shape (times m C_d / H^d later)
// In 3D jd0 = (u, rho) and jd1 = (v, p): the pair weight is 1 / rho_j, and the constants m and
// -56/3 kG of V_j gW are left to the end of the sum, which saves registers and with
// them a wavefront in flight (262,144 particles, 8 lanes: 212 us, against 231 with V_j gW formed per
// pair).  In 2D jd0 = (u, V, p V) and jd1 = (v, rho, p), and V_j gW is formed per pair.  Two records
// per neighbour either way: the sweep is bound by its gathers, not by arithmetic.  d and r2 are the
// pair vector x_ij and its square.  The particle itself (also in the places past its count) has d = 0,
// equal velocities and densities, and adds exactly zero; a neighbour past the support has t = 0 (and see
// walk_again).  No implicit contraction: the products that are fused are written as fma, so a pair rounds the same in
// every copy of the loop.
template <typename T, int DIM, bool RHOSUM, bool RENORM>
__device__ __forceinline__ void fwd_pair(const PairConst<T>& c, const FwdSelf<T>& K,
                                         const FwdNbr<T, DIM, RENORM>& nb, const T* d, T r2, int self,
                                         FwdAcc<T, DIM>& acc)
{
#pragma clang fp contract(off)
    T vj[3];
    T Vj, pVj, rhoj;
    if (DIM == 3) {
        rhoj = nb.a.w;
        Vj = fast_rcp(rhoj);
        vj[0] = nb.b.x; vj[1] = nb.b.y; vj[2] = nb.b.z; pVj = nb.b.w;
    } else {
        Vj = nb.a.z; pVj = nb.a.w;
        vj[0] = nb.b.x; vj[1] = nb.b.y; rhoj = nb.b.z;
    }
    T ue = (K.v[0] - vj[0]) * d[0];
#pragma unroll
    for (int k = 1; k < DIM; ++k) ue = fma(K.v[k] - vj[k], d[k], ue);
    const T q = fast_sqrt(r2) * c.invH;
    const T t = positive_part(T(1) - q);
    const T t2 = t * t;
    const T t4 = t2 * t2;
    const T inv = fast_rcp(r2 + c.epsH2);
    const T pij = ue * inv;
    T sg = T(0);
    if (RENORM) {
        // V_j (G_i + G_j) . grad_i W_ij of the renormalised diffusion
        const T Gj[3] = {nb.G.x, nb.G.y, nb.G.z};
        sg = (K.G[0] + Gj[0]) * d[0];
#pragma unroll
        for (int k = 1; k < DIM; ++k) sg = fma(K.G[k] + Gj[k], d[k], sg);
    }
    if (DIM == 3) {
        const T g = (Vj * t4) * (t * fma(T(-5), t, T(6)));   // 5 q + 1 = 6 - 5 t
        const T cg = fma(c.cA, pij, -(K.p + pVj)) * g;
#pragma unroll
        for (int k = 0; k < DIM; ++k) acc.ax[k] = fma(cg, d[k], acc.ax[k]);
        acc.rdv = fma(g, ue, acc.rdv);
        acc.rdd = fma((K.rho - rhoj) * (r2 * inv), g, acc.rdd);
        if (RENORM) acc.rdg = fma(g, sg, acc.rdg);
    } else {
        const T gF = c.kGF * (t4 * t * fma(T(5), q, T(1)));  // grad W = gF x_ij
        const T cg = fma(fma(c.cA, pij, -K.p), Vj, -pVj) * gF;
#pragma unroll
        for (int k = 0; k < DIM; ++k) acc.ax[k] = fma(cg, d[k], acc.ax[k]);
        acc.rdv = fma(Vj, gF * ue, acc.rdv);
        acc.rdd = fma(Vj * (K.rho - rhoj), gF * r2 * inv, acc.rdd);
        if (RENORM) acc.rdg = fma(Vj, gF * sg, acc.rdg);
    }
    if (RHOSUM) {
        const T w6 = nb.j != self ? t4 * t2 : T(0);   // its own W(0) = 1 is in the sum from the start
        acc.rs = fma(w6, fma(q, fma(q, T(35.0 / 3.0), T(6)), T(1)), acc.rs);
    }
}

// Cell assignment of the next step's sort, done by the sweep that produced the positions
// (same arithmetic as k_assign).  Null cell_count: no sort follows.
struct NextCells {
    const int32_t* blk_rank;
    int32_t* cell_count;
    int32_t* cell_of;
    CellMembers members;
};

// LPP lanes share a particle and walk its row with sweep_list; wavefronts whose particles all lie more
// than the support inside the box run a copy of the pair loop without the periodic image (the same
// roundings), 6 of 45 (2D) instructions per pair less.
// Bound: the vector memory path, but no one rate of it.  Of a large launch (512-simulation batch, 3D 64^3)
// the gathers take 56 to 70 % at 17.9 clocks each (64 bytes a clock are 16 for a wavefront's 16-byte gather;
// 17.9 measured where quads of lanes read consecutive records, as list positions mostly do), the vector
// L1's lines 73 to 77 % at one a clock, and vector issue 54 to 57 %; the data return is busy 89 to 94 %, two
// fifths of that waiting for the L1.  What is left is latency at four to six wavefronts per SIMD: more
// gathers in flight helped, a quarter fewer vector instructions changed little by themselves.  Small launches are bound by a wavefront's own chain.  Measured, before
// (a load per list entry, a test of every position against the count and of every pair against the
// support) and now: 2D 32^2 FP64 13.5 and 8.9 us, 2D 101^2 8.2 and 7.1, 2D 256^2 15.0 and 13.7, 3D 47^3
// 86.5 and 83.0, 3D 64^3 222 and 213, 3D 20^3 FP64 27.3 and 20.7, 512-simulation batch 335 and 328.
// Registers: 80 in FP32 2D, six wavefronts per SIMD (one more register costs the batch 3 %), hence the
// 32-bit indices.
// Copying a workgroup's reach to LDS first (10 to 12 clocks a gather) took twice as long: the copy's 39 to 58
// KB leave too few wavefronts per CU.
template <typename T, int DIM, int MODE, int LPP, bool RENORM>
__global__ __launch_bounds__((kSweepThreads<T, DIM, LPP>))
void k_sweep(int64_t N, int32_t width, const int32_t* __restrict__ nbr,
                                               const int32_t* __restrict__ nbr_count,
                                               const vec4_t<T>* __restrict__ jd0, const vec4_t<T>* __restrict__ jd1,
                                               StatePtrs<T, DIM> cur, StatePtrs<T, DIM> dst,
                                               const int32_t* __restrict__ orig, T* __restrict__ drho_out,
                                               T* __restrict__ acc_out, T* __restrict__ rhosum_out,
                                               const int32_t* __restrict__ psim,
                                               const SimConst<T>* __restrict__ sims, int32_t* __restrict__ status,
                                               NextCells next, NextSlot<T> ns,
                                               unsigned long long* __restrict__ pair_counter,
                                               const vec4_t<T>* __restrict__ jdG)
{
    constexpr int NQ = kLeaves / LPP;
    static_assert(LPP == 2 || LPP == 4 || LPP == 8, "lanes per particle must be 2, 4 or 8");
    const uint32_t t = (uint32_t)xcd_remap(blockIdx.x, gridDim.x) * blockDim.x + threadIdx.x;
    const uint32_t i = t / LPP;   // N records fit 32-bit offsets
    const int r = (int)(t % LPP);
    int accepted = 0;  // listed pairs with r < H (lists with a skin)
    if (i < N) {
        const int s = sim_of(psim, i);
        FwdAcc<T, DIM> acc[NQ];
        const PairConst<T> c = pair_const_of(sims, s);
        auto load_self = [&](uint32_t i0, FwdSelf<T>& K0) {
            const vec4_t<T> a = jd0[i0], b = jd1[i0];
            K0.u[2] = K0.v[2] = T(0);
            unpack_u<T, DIM>(a, K0.u);
            K0.v[0] = b.x;
            K0.v[1] = b.y;
            if (DIM == 3) K0.v[2] = b.z;
            K0.rho = (DIM == 3) ? a.w : b.z;
            K0.p = b.w;
            K0.G[0] = K0.G[1] = K0.G[2] = T(0);
            if (RENORM) {
                const vec4_t<T> g = jdG[i0];
                K0.G[0] = g.x;
                K0.G[1] = g.y;
                K0.G[2] = g.z;
            }
        };
        FwdSelf<T> K;
        load_self(i, K);
        int n = nbr_count[i];
        n = n < width ? n : width;
        const int32_t* row = nbr + (int64_t)i * width;
        // the particle's own entry and the places past the count, at r2 = 0, are counted by the loop
        if (r == 0 && n > 0) accepted = n - positions_visited<T, LPP>(n, width) - 1;
        auto clear = [&]() {
#pragma unroll
            for (int q = 0; q < NQ; ++q) {
                acc[q].ax[0] = acc[q].ax[1] = acc[q].ax[2] = T(0);
                acc[q].rdv = acc[q].rdd = acc[q].rs = acc[q].rdg = T(0);
            }
            // W(0) = 1 of the particle itself
            if (MODE == kModeRhs && r == 0 && n > 0) acc[0].rs = T(1);
        };
        using Nbr = FwdNbr<T, DIM, RENORM>;
        auto gather = [&](int j, Nbr& nb) {
            nb.j = j;
            nb.a = ldo(jd0, (uint32_t)j);
            nb.b = ldo(jd1, (uint32_t)j);
            if (RENORM) nb.G = ldo(jdG, (uint32_t)j);
        };
        auto pairs = [&](auto image, auto walk) {
            walk([&](int q, Nbr& nb) {
                T d[3];
                const T r2 = pair_vector<T, DIM, decltype(image)::value>(K.u, nb.a, c.L, c.invL, d);
                accepted += r2 < c.H2 ? 1 : 0;
                fwd_pair<T, DIM, MODE == kModeRhs, RENORM>(c, K, nb, d, r2, (int)i, acc[q]);
            });
        };
        auto groups = [&](auto&& pair) { sweep_list<(sizeof(T) == 8), LPP, Nbr>(row, width, n, r, (int)i, gather, pair); };
        auto tail = [&](auto&& pair) { list_tail<LPP, Nbr>(row, width, n, r, (int)i, gather, pair); };
        T ax[3] = {0, 0, 0}, rdv = 0, rdd = 0, rs = 0, rdg = 0;
        auto combine = [&]() -> T {
            constexpr bool kSum = MODE == kModeRhs;
            constexpr int NV = DIM + 2 + (kSum ? 1 : 0) + (RENORM ? 1 : 0);
            T leaf[NV][NQ], out[NV];
#pragma unroll
            for (int q = 0; q < NQ; ++q) {
#pragma unroll
                for (int k = 0; k < DIM; ++k) leaf[k][q] = acc[q].ax[k];
                leaf[DIM][q] = acc[q].rdv;
                leaf[DIM + 1][q] = acc[q].rdd;
                if (kSum) leaf[DIM + 2][q] = acc[q].rs;
                if (RENORM) leaf[NV - 1][q] = acc[q].rdg;
            }
            combine_leaves<LPP, NV>(leaf, out);
#pragma unroll
            for (int k = 0; k < DIM; ++k) ax[k] = out[k];
            rdv = out[DIM];
            rdd = out[DIM + 1];
            if (kSum) rs = out[DIM + 2];
            if (RENORM) rdg = out[NV - 1];
            T sum = T(0);
#pragma unroll
            for (int v = 0; v < NV; ++v) sum += fabs(out[v]);
            return sum;
        };
        clear();
        if (wave_inside<T, DIM>(K.u, c.H, c.L)) pairs(std::false_type{}, groups);
        else pairs(std::true_type{}, groups);
        pairs(std::true_type{}, tail);
        if (__builtin_expect(!isfinite(combine()), 0) && past_support(sims[s])) {
            const uint32_t i2 = opaque(i);
            const PairConst<T> c2 = pair_const(sims[opaque(s)]);
            FwdSelf<T> K2;
            load_self(i2, K2);
            clear();
            walk_again<LPP, Nbr>(nbr + (int64_t)i2 * width, width, nbr_count[i2], r, gather, [&](int q, Nbr& nb) {
                T d[3];
                const T r2 = r2_exact<T, DIM>(K2.u, nb.a, c2.L, c2.invL, d);
                if (r2 < c2.H2) fwd_pair<T, DIM, MODE == kModeRhs, RENORM>(c2, K2, nb, d, r2, (int)i2, acc[q]);
            });
            combine();
        }
        if (r == 0) {
            const SimConst<T>& S = sims[s];
            if (DIM == 3) {
                // the constants that the 3D pair terms leave out (V_j gW = scale g)
                const T scale = S.kG * T(-56.0 / 3.0) * S.m;
#pragma unroll
                for (int k = 0; k < DIM; ++k) ax[k] = scale * ax[k];
                rdv = scale * rdv;
                rdd = scale * rdd;
                rdg = scale * rdg;
            }
            const T invrho = fast_rcp(K.rho);
            T a[3];
#pragma unroll
            for (int k = 0; k < DIM; ++k) a[k] = ax[k] * invrho;
            // renormalised diffusion: -delta H c0 sum_j V_j (G_i + G_j) . grad_i W_ij, cD = 2 delta H c0
            const T drho = RENORM ? K.rho * rdv + S.cD * rdd - T(0.5) * S.cD * rdg : K.rho * rdv + S.cD * rdd;
            if (MODE == kModeStep) {
                bool bad = !isfinite(drho);
                const T dt = S.dt;
                int cc[3] = {0, 0, 0};
                T xn[3] = {0, 0, 0}, vn[3] = {0, 0, 0};
#pragma unroll
                for (int k = 0; k < DIM; ++k) {
                    vn[k] = K.v[k] + dt * a[k];
                    xn[k] = cur.x[k][i] + dt * vn[k];
                    dst.v[k][i] = vn[k];
                    dst.x[k][i] = xn[k];
                    bad = bad || !isfinite(vn[k]) || !isfinite(xn[k]);
                    cc[k] = cell_coord(wrap_pos(isfinite(xn[k]) ? xn[k] : T(0), S.L, S.invL), S.cinv, S.nc);
                }
                const T rhon = K.rho + dt * drho;
                dst.rho[i] = rhon;
                if (bad) atomicOr(&status[s], kFlagNonfinite);
                if (next.cell_count) {
                    const int gcell = global_cell<T, DIM>(S, next.blk_rank, cc[0], cc[1], cc[2]);
                    next.cell_of[i] = gcell;
                    add_member(next.members, gcell, atomicAdd(&next.cell_count[gcell], 1), (int32_t)i, orig[i]);
                }
                if (ns.jd0) {
                    // packed records of the next step, as the sort would write them
                    T u[3] = {0, 0, 0};
#pragma unroll
                    for (int k = 0; k < DIM; ++k) u[k] = wrap_pos(isfinite(xn[k]) ? xn[k] : T(0), S.L, S.invL);
                    const T V = S.m * fast_rcp(rhon);
                    const T pn = tait(S, rhon);
                    const T pV = pn * V;
                    vec4_t<T> pa, pb;
                    if (DIM == 3) {
                        pa.x = u[0]; pa.y = u[1]; pa.z = u[2]; pa.w = rhon;
                        pb.x = vn[0]; pb.y = vn[1]; pb.z = vn[2]; pb.w = pn;
                    } else {
                        pa.x = u[0]; pa.y = u[1]; pa.z = V; pa.w = pV;
                        pb.x = vn[0]; pb.y = vn[1]; pb.z = rhon; pb.w = pn;
                    }
                    ns.jd0[i] = pa;
                    ns.jd1[i] = pb;
                    ns.orig[i] = orig[i];
                    // displacement since the lists were built (minimum image)
                    const vec4_t<T> ref = ns.uref[i];
                    const T rr[3] = {ref.x, ref.y, ref.z};
                    T d2 = T(0);
#pragma unroll
                    for (int k = 0; k < DIM; ++k) {
                        T d = u[k] - rr[k];
                        d -= S.L * rint(d * S.invL);
                        d2 += d * d;
                    }
                    if (!(d2 <= ref.w * ref.w)) atomicOr(&status[s], kFlagSkin);
                }
            } else {
                const int o = orig[i];
                drho_out[o] = drho;
#pragma unroll
                for (int k = 0; k < DIM; ++k) acc_out[(int64_t)k * N + o] = a[k];
                if (rhosum_out) rhosum_out[o] = S.m * S.kW * rs;
            }
        }
    }
    if (pair_counter) {
        // wave total of the filtered pairs, one integer atomic per wavefront
        int w = accepted;
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) w += __shfl_xor(w, o, 64);
        if ((threadIdx.x & 63) == 0 && w)
            atomicAdd(&pair_counter[(blockIdx.x & (kPairSlots - 1)) * kPairStride], (unsigned long long)w);
    }
}

// ---------------------------------------------------------------- density-summation adjoint
//
// Cotangent of the positions for cotangents g of the summation density rho_i = m sum_j W_ij
// (the backward benchmark of Sec. 4.1): xbar_k = m sum_{j != k} (g_k + g_j) grad_k W_kj, since
// x_k enters k's own sum and, through W_jk = W_kj, every neighbour's.  The self entry of the
// list has a zero pair vector and adds nothing.  Same list traversal and canonical partial
// sums as the forward sweep.

template <typename T>
__global__ __launch_bounds__(256) void k_gather_sorted(int64_t N, const T* __restrict__ in,
                                                       const int32_t* __restrict__ orig, T* __restrict__ out)
{
    const int64_t q = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (q < N) out[q] = in[orig[q]];
}

template <typename T>
struct DensNbr {
    vec4_t<T> a;
    T g;
    __device__ __forceinline__ void keep()
    {
        pin(a);
        asm volatile("" : "+v"(g));
    }
};

template <typename T, int DIM, int LPP>
__global__ __launch_bounds__(256) void k_density_adj(int64_t N, int32_t width, const int32_t* __restrict__ nbr,
                                                     const int32_t* __restrict__ nbr_count,
                                                     const vec4_t<T>* __restrict__ jd0, const T* __restrict__ gs,
                                                     const int32_t* __restrict__ orig,
                                                     const int32_t* __restrict__ psim,
                                                     const SimConst<T>* __restrict__ sims, T* __restrict__ xbar)
{
    constexpr int NQ = kLeaves / LPP;
    static_assert(LPP == 2 || LPP == 4 || LPP == 8, "lanes per particle must be 2, 4 or 8");
    const int64_t t = (int64_t)xcd_remap(blockIdx.x, gridDim.x) * blockDim.x + threadIdx.x;
    const int64_t i = t / LPP;
    const int r = (int)(t - i * LPP);
    if (i >= N) return;
    const SimConst<T>& S = sims[psim[i]];
    const PairConst<T> c = pair_const(S);
    T ui[3] = {0, 0, 0};
    unpack_u<T, DIM>(jd0[i], ui);
    const T gi = gs[i];
    int n = nbr_count[i];
    n = n < width ? n : width;
    const int32_t* row = nbr + i * (int64_t)width;
    T acc[NQ][3];
    auto gather = [&](int j, DensNbr<T>& nb) {
        nb.a = ldo(jd0, (uint32_t)j);
        nb.g = ldo(gs, (uint32_t)j);
    };
    auto clear = [&]() {
#pragma unroll
        for (int q = 0; q < NQ; ++q) acc[q][0] = acc[q][1] = acc[q][2] = T(0);
    };
    auto pairs = [&](auto image, auto within, auto walk) {
        walk([&](int q, DensNbr<T>& nb) {
            T d[3] = {0, 0, 0};
            const T r2 = pair_vector<T, DIM, decltype(image)::value>(ui, nb.a, c.L, c.invL, d);
            if (decltype(within)::value && !(r2 < c.H2)) return;
            const T tt = kernel_t(r2, c.invH);
            const T t2 = tt * tt;
            const T w = (gi + nb.g) * ((t2 * t2) * (tt * fma(T(-5), tt, T(6))));
#pragma unroll
            for (int k = 0; k < DIM; ++k) acc[q][k] = fma(w, d[k], acc[q][k]);
        });
    };
    auto groups = [&](auto&& pair) { sweep_list<(sizeof(T) == 8), LPP, DensNbr<T>>(row, width, n, r, (int)i, gather, pair); };
    auto tail = [&](auto&& pair) { list_tail<LPP, DensNbr<T>>(row, width, n, r, (int)i, gather, pair); };
    T out[3] = {0, 0, 0};
    T tmp[NQ];
    auto combine = [&]() -> T {
        T sum = T(0);
#pragma unroll
        for (int k = 0; k < DIM; ++k) {
#pragma unroll
            for (int q = 0; q < NQ; ++q) tmp[q] = acc[q][k];
            out[k] = combine_leaves<LPP>(tmp);
            sum += fabs(out[k]);
        }
        return sum;
    };
    clear();
    if (wave_inside<T, DIM>(ui, S.H, S.L)) pairs(std::false_type{}, std::false_type{}, groups);
    else pairs(std::true_type{}, std::false_type{}, groups);
    pairs(std::true_type{}, std::false_type{}, tail);
    if (__builtin_expect(!isfinite(combine()), 0) && past_support(S)) {
        clear();
        pairs(std::true_type{}, std::true_type{},
              [&](auto&& pair) { walk_again<LPP, DensNbr<T>>(row, width, n, r, gather, pair); });
        combine();
    }
    if (r != 0) return;
    const int o = orig[i];
#pragma unroll
    for (int k = 0; k < DIM; ++k) xbar[(int64_t)k * N + o] = (S.m * c.kGF) * out[k];
}

// ---------------------------------------------------------------- explicit Runge-Kutta stages

// out = s0 base + sum_j c[j] K[j] over every field of the states (original order), with up to
// four terms; out may be base (every element is read before it is written).  s0 and the c[j]
// are multiplied by the particle's simulation time step when s0_dt / c_dt are set.  Stage
// states u_i = u + dt sum_j A_ij k_j, the step's end u + dt sum_i b_i k_i, and the adjoint's
// stage cotangents are all of this form.
constexpr int kMaxStages = 4;

template <typename T, int DIM>
struct LinComb {
    StatePtrs<T, DIM> out, base;
    T s0;
    int s0_dt, c_dt, nterm;
    T c[kMaxStages];
    StatePtrs<T, DIM> K[kMaxStages];
};

template <typename T, int DIM>
__device__ __forceinline__ void lincomb_at(const LinComb<T, DIM>& L, int64_t i, T dt, T* x, T* v, T& r)
{
    const T s0 = L.s0_dt ? L.s0 * dt : L.s0;
#pragma unroll
    for (int k = 0; k < DIM; ++k) {
        x[k] = s0 * L.base.x[k][i];
        v[k] = s0 * L.base.v[k][i];
    }
    r = s0 * L.base.rho[i];
    for (int j = 0; j < L.nterm; ++j) {
        const T c = L.c_dt ? L.c[j] * dt : L.c[j];
#pragma unroll
        for (int k = 0; k < DIM; ++k) {
            x[k] += c * L.K[j].x[k][i];
            v[k] += c * L.K[j].v[k][i];
        }
        r += c * L.K[j].rho[i];
    }
#pragma unroll
    for (int k = 0; k < DIM; ++k) {
        L.out.x[k][i] = x[k];
        L.out.v[k][i] = v[k];
    }
    L.out.rho[i] = r;
}

template <typename T, int DIM>
__global__ __launch_bounds__(256) void k_lincomb(int64_t N, LinComb<T, DIM> L, const int32_t* __restrict__ psim,
                                                 const SimConst<T>* __restrict__ sims)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= N) return;
    T x[3], v[3], r;
    lincomb_at<T, DIM>(L, i, sims[sim_of(psim, i)].dt, x, v, r);
}

// A stage state formed (in original order, for the later stages and the adjoint) and put into the slot
// whose lists it keeps, in one pass.  Bound: launch and memory latency (2D 151^2: 3.9 us; as k_lincomb and
// k_repack, two launches of 3.5).
template <typename T, int DIM>
__global__ __launch_bounds__(256) void k_stage_state(int64_t N, LinComb<T, DIM> L, StageSlot<T, DIM> slot,
                                                     const int32_t* __restrict__ psim,
                                                     const SimConst<T>* __restrict__ sims,
                                                     int32_t* __restrict__ status)
{
    const int64_t d = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (d >= N) return;
    const int s = sim_of(psim, d);
    const SimConst<T>& S = sims[s];
    T x[3] = {0, 0, 0}, v[3] = {0, 0, 0}, r;
    lincomb_at<T, DIM>(L, slot.orig[d], S.dt, x, v, r);
    put_stage<T, DIM>(slot, d, S, x, v, r, &status[s]);
}

// dst = src, every field: one launch (2D 151^2: 3.6 us), where a copy per array took 2 D + 1 of 2.2 and the
// gaps between them.
template <typename T, int DIM>
__global__ __launch_bounds__(256) void k_copy_state(int64_t N, StatePtrs<T, DIM> src, StatePtrs<T, DIM> dst)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= N) return;
#pragma unroll
    for (int k = 0; k < DIM; ++k) {
        dst.x[k][i] = src.x[k][i];
        dst.v[k][i] = src.v[k][i];
    }
    dst.rho[i] = src.rho[i];
}

// ---------------------------------------------------------------- symplectic Euler
//
// DualSPHysics' symplectic scheme (Sec. 3.4, App. C), h = dt/2: the predictor state
// u_h = (x + h v, v + h a1, rho + h D1) is formed by k_lincomb, the corrector's rates
// (a2, D2) = f(u_h) by a right-hand-side sweep, and the step ends with
//   v' = v + dt a2,  x' = x_h + h v',  rho' = rho (2 - e) / (2 + e),  e = -dt D2 / rho_h.
// All three kernels run in original particle order.

// The corrector, u in place; uh = predictor state, r2 = (., a2, D2).
template <typename T, int DIM>
__global__ __launch_bounds__(256) void k_symp_final(int64_t N, StatePtrs<T, DIM> u, StatePtrs<T, DIM> uh,
                                                    StatePtrs<T, DIM> r2, const int32_t* __restrict__ psim,
                                                    const SimConst<T>* __restrict__ sims)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= N) return;
    const T dt = sims[psim[i]].dt;
    const T h = T(0.5) * dt;
#pragma unroll
    for (int k = 0; k < DIM; ++k) {
        const T vn = u.v[k][i] + dt * r2.v[k][i];
        u.v[k][i] = vn;
        u.x[k][i] = uh.x[k][i] + h * vn;
    }
    const T e = -dt * r2.rho[i] / uh.rho[i];
    u.rho[i] = u.rho[i] * (T(2) - e) / (T(2) + e);
}

// Transpose of the corrector.  cot = (xb', vb', rb') of u'; cb (null for none) = cotangent of
// (a2, D2) where the next step re-uses them.  With vt = vb' + h xb', g(e) = (2 - e)/(2 + e),
// eb = rb' rho g'(e):
//   kb2 = (0, dt vt + cb_a, -dt eb / rho_h + cb_D)       rates' cotangent, for the VJP at u_h
//   uhd = (xb', 0, eb dt D2 / rho_h^2)                    u_h's cotangent outside that VJP
//   b0  = (0, vt, rb' g)                                  u's cotangent outside the predictor
template <typename T, int DIM>
__global__ __launch_bounds__(256) void k_symp_final_adj(int64_t N, StatePtrs<T, DIM> cot, const T* __restrict__ rho,
                                                        const T* __restrict__ rho_h, const T* __restrict__ d2,
                                                        StatePtrs<T, DIM> cb, int has_cb, StatePtrs<T, DIM> kb2,
                                                        StatePtrs<T, DIM> uhd, StatePtrs<T, DIM> b0,
                                                        const int32_t* __restrict__ psim,
                                                        const SimConst<T>* __restrict__ sims)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= N) return;
    const T dt = sims[psim[i]].dt;
    const T h = T(0.5) * dt;
#pragma unroll
    for (int k = 0; k < DIM; ++k) {
        const T xb = cot.x[k][i];
        const T vt = cot.v[k][i] + h * xb;
        kb2.x[k][i] = T(0);
        kb2.v[k][i] = dt * vt + (has_cb ? cb.v[k][i] : T(0));
        uhd.x[k][i] = xb;
        uhd.v[k][i] = T(0);
        b0.x[k][i] = T(0);
        b0.v[k][i] = vt;
    }
    const T rb = cot.rho[i], rh = rho_h[i], D2 = d2[i];
    const T e = -dt * D2 / rh;
    const T g = (T(2) - e) / (T(2) + e);
    const T gp = T(-4) / ((T(2) + e) * (T(2) + e));
    const T eb = rb * rho[i] * gp;
    kb2.rho[i] = -dt * eb / rh + (has_cb ? cb.rho[i] : T(0));
    uhd.rho[i] = eb * dt * D2 / (rh * rh);
    b0.rho[i] = rb * g;
}

// Transpose of the predictor when its rates were re-used (not evaluated from u): with
// kb1 = h ubar_h, u's cotangent is b0 + (0, kb1_x, 0) (the x-rate of the predictor is v) and
// the re-used rates receive (kb1_v, kb1_rho).
template <typename T, int DIM>
__global__ __launch_bounds__(256) void k_symp_pred_adj(int64_t N, StatePtrs<T, DIM> b0, StatePtrs<T, DIM> kb1,
                                                       StatePtrs<T, DIM> cot, StatePtrs<T, DIM> cb)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= N) return;
#pragma unroll
    for (int k = 0; k < DIM; ++k) {
        cot.x[k][i] = b0.x[k][i];
        cot.v[k][i] = b0.v[k][i] + kb1.x[k][i];
        cb.v[k][i] = kb1.v[k][i];
    }
    cot.rho[i] = b0.rho[i];
    cb.rho[i] = kb1.rho[i];
}

// ---------------------------------------------------------------- unsort

template <typename T, int DIM>
__global__ __launch_bounds__(256) void k_unsort(int64_t N, StatePtrs<T, DIM> src, const int32_t* __restrict__ orig,
                                                StatePtrs<T, DIM> dst)
{
    int64_t q = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (q >= N) return;
    const int o = orig[q];
#pragma unroll
    for (int k = 0; k < DIM; ++k) {
        dst.x[k][o] = src.x[k][q];
        dst.v[k][o] = src.v[k][q];
    }
    dst.rho[o] = src.rho[q];
}

// ---------------------------------------------------------------- adjoint

// A particle's adjoint record: (abar, rbar rho) in 3D, (abar, rbar rho, rbar rho^2) in 2D.
template <typename T, int DIM>
__device__ __forceinline__ vec4_t<T> adjoint_record(const T* ab, T rb, T rho)
{
    const T rbr = rb * rho;
    vec4_t<T> a;
    a.x = ab[0];
    a.y = ab[1];
    a.z = (DIM == 3) ? ab[2] : rbr;
    a.w = (DIM == 3) ? rbr : rbr * rho;
    return a;
}

// Gathers the output cotangents into sorted order, with vt = v'_bar + dt x'_bar, abar = dt vt,
// rbar = dt rho'_bar.
template <typename T, int DIM>
__global__ __launch_bounds__(256) void k_adj_prologue(int64_t N, const int32_t* __restrict__ orig,
                                                      StatePtrs<T, DIM> cot, StatePtrs<T, DIM> cur,
                                                      vec4_t<T>* __restrict__ jdA,
                                                      const int32_t* __restrict__ psim,
                                                      const SimConst<T>* __restrict__ sims, int vjp)
{
    int64_t q = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (q >= N) return;
    const SimConst<T>& S = sims[psim[q]];
    const int o = orig[q];
    T ab[3] = {0, 0, 0};
    T rb;
    if (vjp) {
        // the update function's VJP: cot holds the cotangents (kx, ka, krho) of (v, a, drho/dt)
#pragma unroll
        for (int k = 0; k < DIM; ++k) ab[k] = cot.v[k][o];
        rb = cot.rho[o];
    } else {
        // one semi-implicit Euler step: abar = dt (vbar' + dt xbar'), rbar = dt rhobar'
#pragma unroll
        for (int k = 0; k < DIM; ++k) ab[k] = S.dt * (cot.v[k][o] + S.dt * cot.x[k][o]);
        rb = S.dt * cot.rho[o];
    }
    jdA[q] = adjoint_record<T, DIM>(ab, rb, cur.rho[q]);
}

// A stage's cotangent formed (in original order, for the sweep that follows and the earlier stages), its
// adjoint record, and, unless the slot holds it already, the stage's state put into the slot, in one pass
// (2D 151^2: 4.3 us; as k_lincomb, k_repack and k_adj_prologue, three launches of 3.5, 3.5 and 2.8).
template <typename T, int DIM>
__global__ __launch_bounds__(256) void k_stage_cot(int64_t N, LinComb<T, DIM> L, StatePtrs<T, DIM> src,
                                                   StageSlot<T, DIM> slot, vec4_t<T>* __restrict__ jdA,
                                                   const int32_t* __restrict__ psim,
                                                   const SimConst<T>* __restrict__ sims, int32_t* __restrict__ status)
{
    const int64_t d = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (d >= N) return;
    const int s = sim_of(psim, d);
    const SimConst<T>& S = sims[s];
    const int p = slot.orig[d];
    T kx[3], kv[3] = {0, 0, 0}, kr;
    lincomb_at<T, DIM>(L, p, S.dt, kx, kv, kr);
    const T rho = src.rho[p];
    if (slot.jd0) {
        T x[3] = {0, 0, 0}, v[3] = {0, 0, 0};
#pragma unroll
        for (int k = 0; k < DIM; ++k) {
            x[k] = src.x[k][p];
            v[k] = src.v[k][p];
        }
        put_stage<T, DIM>(slot, d, S, x, v, rho, &status[s]);
    }
    jdA[d] = adjoint_record<T, DIM>(kv, kr, rho);
}

// What the adjoint sweep of step t prepares for the adjoint of step t - 1 when both states share
// the particle order (a step within one list-reuse interval), or when the sort of state t has kept each
// particle's place in the order before it (`before`): the prologue records of step t - 1 at the particle's
// index there, from the cotangents the sweep has just formed (null jdA: none).
template <typename T>
struct NextAdj {
    vec4_t<T>* jdA;
    const T* rho;   // densities of state t - 1, sorted order
    const int32_t* before;   // null: the same order
};

template <typename T, int DIM>
struct AdjAcc {
    T gx[3], gv[3];
    T s1, s2;  // the density cotangent is -dp/drho s1 - s2 / rho
    T Gb[3];   // cotangent of the renormalised density gradient
};

// Per-particle adjoint record of a neighbour: jd0 = (u, rho), jd1 = (v, p), jdA = (abar, rbar rho) in
// 3D; jd0 = (u, V, p V), jd1 = (v, rho, p), jdA = (abar, rbar rho, rbar rho^2) in 2D.  They hold
// everything a neighbour contributes: three records per neighbour, and no others for the particle.
template <typename T, int DIM, bool RENORM>
struct AdjNbr {
    vec4_t<T> a, b, A, G;
    __device__ __forceinline__ void keep()
    {
        pin<DIM == 3 ? 4 : 3>(a);
        pin(b);
        pin(A);
        if (RENORM) pin<3>(G);
    }
};

// (four records per neighbour: held, they cost 2D more than the wait; 32^2 FP64 13.2 us against 11.5)
template <typename T, int DIM>
constexpr bool kGatherFirst<AdjNbr<T, DIM, true>> = false;

// Adjoint pair terms, gather form.  For particle k and a neighbour j != k: the partial
// derivatives, with respect to k's position, velocity and density, of the two directed pair
// terms (k,j) and (j,k) contracted with their particles' cotangents (abar, rbar).  With
// e = x_kj, u = v_kj, the kernel gradient gF e and Hessian Jg = gF I + hF e e^T, inv = 1/(r^2+eps H^2),
// pi = (u.e) inv, s = gF r^2 inv, sigma = inv (2 gF + hF r^2 - 2 s), X = cA pi - p_k - p_j, and the
// symmetric weight Phi = V_k V_j / m = m / (rho_k rho_j), every partial has the factor Phi, because
// V_j / rho_k = V_k / rho_j = Phi.  With da = abar_k - abar_j, Q = rbar rho, R = rbar rho^2:
//   B    = cA inv gF (da.e)
//   xbar = Phi [ (B + gF (R_k + R_j)) u + gF X da
//                + (hF (X (da.e) + (R_k + R_j)(u.e)) - 2 pi B + cD sigma (rho_k - rho_j)(Q_k - Q_j)) e ]
//   vbar = Phi (B + gF (R_k + R_j)) e
//   rbar = Phi [ -gF (da.e) (p'_k + X / rho_k) + (gF u.e + cD s)(R_k - R_j) / rho_k ]
// The differences da, u, e, R_k - R_j vanish exactly for the particle itself, whose pair (also in
// the places past its count) therefore adds exactly zero.  V_j is a factor of gF and hF here (1 / rho_j
// in 3D); the particle's own factor of Phi and the constant kGF are applied at the end.
//
// With RENORM, the renormalised diffusion T_i = c sum_j V_j (G_i + G_j) . grad_i W_ij
// (c = -delta H c0) adds, with the gradients held fixed and s = G_k + G_j: xbar += Phi c (Q_k - Q_j) Jg s,
// Gbar += Phi c (Q_k - Q_j) gF e, rbar += Phi c Q_j gF s.e / rho_k.
//
// Bound: as in k_sweep (reads 53 to 71 %, L1 lines 72 to 88 %, vector issue 63 to 70 % of a large launch), three
// records per neighbour.  Dropping the second adjoint record
// (u and the density are in jd0 and jd1), the common factor Phi (62 vector instructions per pair, 80 before) and
// the walk of the rows: 2D 101^2 9.4 and 9.1 us, 2D 256^2 18.4 and 17.2, 3D 47^3 140 and 125, 3D 64^3 318 and
// 318, 3D 20^3 FP64 25.9 and 22.1, 512-simulation batch 439 and 407; with renormalisation, the second pass
// (k_renorm_adj, 3D 32^3) 42.8 and 25.1.
template <typename T>
struct AdjSelf {
    T v[3], a[3];   // velocity, abar
    T rho, p, Q, R;
    T G[3];
};

template <typename T, int DIM, bool RENORM>
__device__ __forceinline__ void adj_pair(const PairConst<T>& c, const AdjSelf<T>& K, const AdjNbr<T, DIM, RENORM>& nb,
                                         const T* e, T r2, AdjAcc<T, DIM>& acc)
{
#pragma clang fp contract(off)
    const T Vj = pair_weight<T, DIM>(nb.a);
    const T rhoj = (DIM == 3) ? nb.a.w : nb.b.z;
    const T pj = nb.b.w;
    const T Qj = (DIM == 3) ? nb.A.w : nb.A.z;
    const T Rj = (DIM == 3) ? Qj * rhoj : nb.A.w;
    const T vj[3] = {nb.b.x, nb.b.y, nb.b.z}, aj[3] = {nb.A.x, nb.A.y, nb.A.z};
    T u[3], da[3];
    u[0] = K.v[0] - vj[0];
    da[0] = K.a[0] - aj[0];
    T ue = u[0] * e[0], de = da[0] * e[0];
#pragma unroll
    for (int k = 1; k < DIM; ++k) {
        u[k] = K.v[k] - vj[k];
        da[k] = K.a[k] - aj[k];
        ue = fma(u[k], e[k], ue);
        de = fma(da[k], e[k], de);
    }
    const T t = kernel_t(r2, c.invH);
    const T t2 = t * t;
    const T vt4 = Vj * (t2 * t2);
    const T g = vt4 * (t * fma(T(-5), t, T(6)));
    const T h = c.hc * vt4;
    const T inv = fast_rcp(r2 + c.epsH2);
    const T pij = ue * inv;
    const T s = g * (r2 * inv);
    const T sig = inv * fma(T(2), g - s, h * r2);   // d s / d e = sig e
    const T X = fma(c.cA, pij, -(K.p + pj));
    const T Rs = K.R + Rj, Rd = K.R - Rj, Qd = K.Q - Qj;
    const T gde = g * de;
    const T B = (c.cA * inv) * gde;
    const T cu = fma(g, Rs, B);
    const T gX = g * X;
    const T ew = fma(X, de, Rs * ue);
    const T ce = fma(h, ew, fma(T(-2) * B, pij, sig * ((c.cD * (K.rho - rhoj)) * Qd)));
#pragma unroll
    for (int k = 0; k < DIM; ++k) {
        acc.gx[k] = fma(cu, u[k], fma(gX, da[k], fma(ce, e[k], acc.gx[k])));
        acc.gv[k] = fma(cu, e[k], acc.gv[k]);
    }
    acc.s1 = acc.s1 + gde;
    acc.s2 = fma(gde, X, fma(-fma(c.cD, s, g * ue), Rd, acc.s2));
    if (RENORM) {
        const T cr = T(-0.5) * c.cD;
        const T Gj[3] = {nb.G.x, nb.G.y, nb.G.z};
        T sv[3], es = T(0);
#pragma unroll
        for (int k = 0; k < DIM; ++k) {
            sv[k] = K.G[k] + Gj[k];
            es = fma(e[k], sv[k], es);
        }
        const T qq = cr * Qd, gq = g * qq, hq = (h * qq) * es;
#pragma unroll
        for (int k = 0; k < DIM; ++k) {
            acc.gx[k] = fma(gq, sv[k], fma(hq, e[k], acc.gx[k]));
            acc.Gb[k] = fma(gq, e[k], acc.Gb[k]);
        }
        acc.s2 = fma(-(cr * Qj), g * es, acc.s2);
    }
}

// Wavefronts per SIMD the adjoint sweep's registers are held to: in FP32 2D five (96 registers instead of
// 113: the 512-simulation batch 399 us a launch against 463, although 7 registers spill with four lanes and 4
// with eight), with two lanes four (118 registers: 588 us against 726 and more, where five left 19 to 26 spilt).
// Not in 3D, which spills under it, nor with RENORM (2D 256^2, 64 steps and their adjoint: 8.6 ms with the limit,
// 7.2 without).
template <typename T, int DIM, int LPP, bool RENORM>
constexpr int kAdjWaves = sizeof(T) == 4 && DIM == 2 && !RENORM ? (LPP == 2 ? 4 : 5) : 1;

// Within one list-reuse interval consecutive adjoint sweeps hand the cotangents on in sorted order
// (cin_sorted, cout_sorted): contiguous accesses, where the caller's order scatters them.
template <typename T, int DIM, int LPP, bool RENORM>
__global__ __launch_bounds__((kSweepThreads<T, DIM, LPP>), (kAdjWaves<T, DIM, LPP, RENORM>))
void k_adj_sweep(int64_t N, int32_t width, const int32_t* __restrict__ nbr,
                                                   const int32_t* __restrict__ nbr_count,
                                                   const vec4_t<T>* __restrict__ jd0,
                                                   const vec4_t<T>* __restrict__ jd1,
                                                   const vec4_t<T>* __restrict__ jdA,
                                                   const int32_t* __restrict__ orig, StatePtrs<T, DIM> cin,
                                                   int cin_sorted, StatePtrs<T, DIM> cout, int cout_sorted,
                                                   const int32_t* __restrict__ psim,
                                                   const SimConst<T>* __restrict__ sims, int32_t* __restrict__ status,
                                                   int vjp, const vec4_t<T>* __restrict__ jdG,
                                                   const vec4_t<T>* __restrict__ jdL, vec4_t<T>* __restrict__ gbar,
                                                   NextAdj<T> na)
{
    constexpr int NQ = kLeaves / LPP;
    static_assert(LPP == 2 || LPP == 4 || LPP == 8, "lanes per particle must be 2, 4 or 8");
    const int64_t t = (int64_t)xcd_remap(blockIdx.x, gridDim.x) * blockDim.x + threadIdx.x;
    const int64_t k = t / LPP;
    const int r = (int)(t - k * LPP);
    if (k >= N) return;
    const int s = sim_of(psim, k);
    AdjAcc<T, DIM> acc[NQ];
    const PairConst<T> c = pair_const_of(sims, s);
    auto load_self = [&](int64_t k0, T* u, AdjSelf<T>& K0) {
        const vec4_t<T> a = jd0[k0], b = jd1[k0], A = jdA[k0];
        unpack_u<T, DIM>(a, u);
        K0.v[0] = b.x; K0.v[1] = b.y; K0.v[2] = (DIM == 3) ? b.z : T(0);
        K0.a[0] = A.x; K0.a[1] = A.y; K0.a[2] = (DIM == 3) ? A.z : T(0);
        K0.rho = (DIM == 3) ? a.w : b.z;
        K0.p = b.w;
        K0.Q = (DIM == 3) ? A.w : A.z;
        K0.R = (DIM == 3) ? A.w * a.w : A.w;
        K0.G[0] = K0.G[1] = K0.G[2] = T(0);
        if (RENORM) {
            const vec4_t<T> g = jdG[k0];
            K0.G[0] = g.x;
            K0.G[1] = g.y;
            K0.G[2] = g.z;
        }
    };
    T uk[3] = {0, 0, 0};
    AdjSelf<T> K;
    load_self(k, uk, K);
    int n = nbr_count[k];
    n = n < width ? n : width;
    const int32_t* row = nbr + k * (int64_t)width;
    using Nbr = AdjNbr<T, DIM, RENORM>;
    auto gather = [&](int j, Nbr& nb) {
        nb.a = ldo(jd0, (uint32_t)j);
        nb.b = ldo(jd1, (uint32_t)j);
        nb.A = ldo(jdA, (uint32_t)j);
        if (RENORM) nb.G = ldo(jdG, (uint32_t)j);
    };
    auto clear = [&]() {
#pragma unroll
        for (int q = 0; q < NQ; ++q) {
#pragma unroll
            for (int d = 0; d < 3; ++d) acc[q].gx[d] = acc[q].gv[d] = acc[q].Gb[d] = T(0);
            acc[q].s1 = acc[q].s2 = T(0);
        }
    };
    auto pairs = [&](auto image, auto walk) {
        walk([&](int q, Nbr& nb) {
            T e[3];
            const T r2 = pair_vector<T, DIM, decltype(image)::value>(uk, nb.a, c.L, c.invL, e);
            adj_pair<T, DIM, RENORM>(c, K, nb, e, r2, acc[q]);
        });
    };
    // four records per neighbour with RENORM: two pairs at a time, or the registers leave too few wavefronts
    auto groups = [&](auto&& pair) {
        sweep_list<(sizeof(T) == 8 || RENORM), LPP, Nbr>(row, width, n, r, (int)k, gather, pair);
    };
    auto tail = [&](auto&& pair) { list_tail<LPP, Nbr>(row, width, n, r, (int)k, gather, pair); };
    T gx[3] = {0, 0, 0}, gv[3] = {0, 0, 0}, Gb[3] = {0, 0, 0}, s1 = 0, s2 = 0;
    auto combine = [&]() -> T {
        constexpr int NV = (RENORM ? 3 : 2) * DIM + 2;
        T leaf[NV][NQ], out[NV];
#pragma unroll
        for (int q = 0; q < NQ; ++q) {
#pragma unroll
            for (int d = 0; d < DIM; ++d) {
                leaf[d][q] = acc[q].gx[d];
                leaf[DIM + d][q] = acc[q].gv[d];
                if (RENORM) leaf[2 * DIM + d][q] = acc[q].Gb[d];
            }
            leaf[NV - 2][q] = acc[q].s1;
            leaf[NV - 1][q] = acc[q].s2;
        }
        combine_leaves<LPP, NV>(leaf, out);
#pragma unroll
        for (int d = 0; d < DIM; ++d) {
            gx[d] = out[d];
            gv[d] = out[DIM + d];
            if (RENORM) Gb[d] = out[2 * DIM + d];
        }
        s1 = out[NV - 2];
        s2 = out[NV - 1];
        T sum = T(0);
#pragma unroll
        for (int v = 0; v < NV; ++v) sum += fabs(out[v]);
        return sum;
    };
    clear();
    if (wave_inside<T, DIM>(uk, c.H, c.L)) pairs(std::false_type{}, groups);
    else pairs(std::true_type{}, groups);
    pairs(std::true_type{}, tail);
    if (__builtin_expect(!isfinite(combine()), 0) && past_support(sims[s])) {
        const int64_t k2 = opaque(k);
        const PairConst<T> c2 = pair_const(sims[opaque(s)]);
        T u2[3] = {0, 0, 0};
        AdjSelf<T> K2;
        load_self(k2, u2, K2);
        clear();
        walk_again<LPP, Nbr>(nbr + k2 * width, width, nbr_count[k2], r, gather, [&](int q, Nbr& nb) {
            T e[3];
            const T r2 = r2_exact<T, DIM>(u2, nb.a, c2.L, c2.invL, e);
            if (r2 < c2.H2) adj_pair<T, DIM, RENORM>(c2, K2, nb, e, r2, acc[q]);
        });
        combine();
    }
    if (r != 0) return;
    const SimConst<T>& S = sims[s];
    // the particle's factor of Phi = m / (rho_k rho_j) and the kernel constant (the neighbour's factor
    // is V_j in 2D, 1 / rho_j in 3D)
    const T rhok = K.rho;
    const T ir = fast_rcp(rhok);
    const T kGF = S.kG * T(-56.0 / 3.0);
    const T scale = (DIM == 3) ? kGF * (S.m * ir) : kGF * ir;
#pragma unroll
    for (int d = 0; d < DIM; ++d) {
        gx[d] = scale * gx[d];
        gv[d] = scale * gv[d];
        Gb[d] = scale * Gb[d];
    }
    const T gr = -scale * fma(tait_slope(S, rhok), s1, ir * s2);
    if (RENORM) {
        // gbar_k = L_k^T Gbar_k (L symmetric), for the second renormalisation pass
        T L[6] = {0, 0, 0, 0, 0, 0};
        if (DIM == 2) {
            const vec4_t<T> l0 = jdL[k];
            L[0] = l0.x; L[1] = l0.y; L[2] = l0.z;
        } else {
            const vec4_t<T> l0 = jdL[2 * k], l1 = jdL[2 * k + 1];
            L[0] = l0.x; L[1] = l0.y; L[2] = l0.z; L[3] = l0.w; L[4] = l1.x; L[5] = l1.y;
        }
        T gb[3];
        sym_mul<T, DIM>(L, Gb, gb);
        vec4_t<T> o4;
        o4.x = gb[0];
        o4.y = gb[1];
        o4.z = gb[2];
        o4.w = T(0);
        gbar[k] = o4;
    }
    const T dt = S.dt;
    const int64_t o = (cin_sorted && cout_sorted) ? k : (int64_t)orig[k];
    const int64_t ci = cin_sorted ? k : o, co = cout_sorted ? k : o;
    bool bad = !isfinite(gr);
    T xn[3] = {0, 0, 0}, vn[3] = {0, 0, 0};
#pragma unroll
    for (int d = 0; d < DIM; ++d) {
        const T xb = cin.x[d][ci];
        const T vb = cin.v[d][ci];
        if (vjp) {
            // (xbar, vbar, rhobar) = (J_x^T, kx + J_v^T, J_rho^T): dx/dt = v adds kx to vbar
            xn[d] = gx[d];
            vn[d] = xb + gv[d];
        } else {
            xn[d] = xb + gx[d];
            vn[d] = vb + dt * xb + gv[d];
        }
        cout.x[d][co] = xn[d];
        cout.v[d][co] = vn[d];
        bad = bad || !isfinite(gx[d]) || !isfinite(gv[d]);
    }
    const T rn = vjp ? gr : cin.rho[ci] + gr;
    cout.rho[co] = rn;
    if (bad) atomicOr(&status[s], kFlagNonfinite);
    if (na.jdA) {
        // the prologue of the previous step's adjoint (same arithmetic as k_adj_prologue)
        T ab[3] = {0, 0, 0};
#pragma unroll
        for (int d = 0; d < DIM; ++d) ab[d] = dt * (vn[d] + dt * xn[d]);
        const T rb = dt * rn;
        const uint32_t q = na.before ? (uint32_t)na.before[k] : k;   // index in state t - 1
        na.jdA[q] = adjoint_record<T, DIM>(ab, rb, na.rho[q]);
    }
}

// Second pass of the renormalised diffusion's adjoint: the cotangents of the moment sums
// M_i, g_i (Mbar_i = -gbar_i G_i^T, gbar_i = L_i Gbar_i from the adjoint sweep) carried to
// positions and densities, gathered over each particle's own sums and its neighbours':
//   own (e = x_k - x_j, w = gF e, Jg v = gF v + hF (e.v) e):
//     xbar_k += V_j [gbar_k (G_k.w) + Jg G_k (gbar_k.e)] + V_j (rho_j - rho_k) Jg gbar_k
//     rbar_k -= V_j (gbar_k.w)
//   neighbour's:
//     xbar_k += V_k [gbar_j (G_j.w) + Jg G_j (gbar_j.e)] - V_k (rho_k - rho_j) Jg gbar_j
//     rbar_k += -V_k (gbar_j.w) + (V_k / rho_k) [(rho_k - rho_j)(gbar_j.w) - (e.gbar_j)(G_j.w)]
// added to the cotangents (original order).  Same list traversal and partial sums.
template <typename T>
struct RenormAdjSelf {
    T u[3], G[3], b[3];   // position, G_k, gbar_k
    T V, rho, ir;
};

template <typename T, int DIM>
struct RenormAdjNbr {
    vec4_t<T> a, b, G, gb;
    __device__ __forceinline__ void keep()
    {
        pin<DIM == 3 ? 4 : 3>(a);
        if (DIM == 2) pin<3>(b);
        pin<3>(G);
        pin<3>(gb);
    }
};

template <typename T, int DIM, int LPP>
__global__ __launch_bounds__(256) void k_renorm_adj(int64_t N, int32_t width, const int32_t* __restrict__ nbr,
                                                    const int32_t* __restrict__ nbr_count,
                                                    const vec4_t<T>* __restrict__ jd0, const vec4_t<T>* __restrict__ jd1,
                                                    const vec4_t<T>* __restrict__ jdG,
                                                    const vec4_t<T>* __restrict__ gbar,
                                                    const int32_t* __restrict__ orig, StatePtrs<T, DIM> cot,
                                                    const int32_t* __restrict__ psim,
                                                    const SimConst<T>* __restrict__ sims)
{
    constexpr int NQ = kLeaves / LPP;
    const int64_t t = (int64_t)xcd_remap(blockIdx.x, gridDim.x) * blockDim.x + threadIdx.x;
    const int64_t k = t / LPP;
    const int r = (int)(t - k * LPP);
    if (k >= N) return;
    const SimConst<T>& S = sims[psim[k]];
    const PairConst<T> c = pair_const(S);
    auto load_self = [&](int64_t k0, RenormAdjSelf<T>& K0) {
        const vec4_t<T> a = jd0[k0], g4 = jdG[k0], b4 = gbar[k0];
        K0.u[2] = T(0);
        unpack_u<T, DIM>(a, K0.u);
        K0.V = rec_volume<T, DIM>(a, sims[psim[k0]].m);
        K0.rho = (DIM == 3) ? a.w : jd1[k0].z;
        K0.ir = T(1) / K0.rho;
        K0.G[0] = g4.x; K0.G[1] = g4.y; K0.G[2] = g4.z;
        K0.b[0] = b4.x; K0.b[1] = b4.y; K0.b[2] = b4.z;
    };
    RenormAdjSelf<T> K;
    load_self(k, K);
    int n = nbr_count[k];
    n = n < width ? n : width;
    const int32_t* row = nbr + k * (int64_t)width;
    T ax[NQ][3], ar[NQ];
    auto clear = [&]() {
#pragma unroll
        for (int q = 0; q < NQ; ++q) ax[q][0] = ax[q][1] = ax[q][2] = ar[q] = T(0);
    };
    using Nbr = RenormAdjNbr<T, DIM>;
    auto gather = [&](int j, Nbr& nb) {
        nb.a = ldo(jd0, (uint32_t)j);
        if (DIM == 2) nb.b = ldo(jd1, (uint32_t)j);
        nb.G = ldo(jdG, (uint32_t)j);
        nb.gb = ldo(gbar, (uint32_t)j);
    };
    auto add = [&](const RenormAdjSelf<T>& K0, T m, T invH, T hc, const Nbr& nb, const T* e, T r2, T* x, T& a) {
        const T tt = kernel_t(r2, invH);
        const T t2 = tt * tt;
        const T t4 = t2 * t2;
        const T g = t4 * (tt * fma(T(-5), tt, T(6)));   // Jg v = kGF (g v + h (e.v) e)
        const T h = hc * t4;
        const T Vj = rec_volume<T, DIM>(nb.a, m);
        const T rhoj = (DIM == 3) ? nb.a.w : nb.b.z;
        const T Gj[3] = {nb.G.x, nb.G.y, nb.G.z}, bj[3] = {nb.gb.x, nb.gb.y, nb.gb.z};
        T bke = K0.b[0] * e[0], bje = bj[0] * e[0], Gke = K0.G[0] * e[0], Gje = Gj[0] * e[0];
#pragma unroll
        for (int d = 1; d < DIM; ++d) {
            Gke = fma(K0.G[d], e[d], Gke);
            bke = fma(K0.b[d], e[d], bke);
            Gje = fma(Gj[d], e[d], Gje);
            bje = fma(bj[d], e[d], bje);
        }
        // own terms carry G_k.e + (rho_j - rho_k), the neighbour's G_j.e + (rho_j - rho_k)
        const T drk = rhoj - K0.rho;
        const T P = Gke + drk, Q = Gje + drk;
        const T vP = Vj * P, vb = Vj * bke, wQ = K0.V * Q, wb = K0.V * bje;
        const T he = h * fma(vb, P, wb * Q);
#pragma unroll
        for (int d = 0; d < DIM; ++d) {
            const T z = fma(K0.b[d], vP, fma(K0.G[d], vb, fma(bj[d], wQ, Gj[d] * wb)));
            x[d] = fma(g, z, fma(he, e[d], x[d]));
        }
        a = fma(-g, fma(wb, fma(K0.ir, Q, T(1)), vb), a);
    };
    auto pairs = [&](auto image, auto walk) {
        walk([&](int q, Nbr& nb) {
            T e[3] = {0, 0, 0};
            const T r2 = pair_vector<T, DIM, decltype(image)::value>(K.u, nb.a, c.L, c.invL, e);
            add(K, S.m, c.invH, c.hc, nb, e, r2, ax[q], ar[q]);
        });
    };
    auto groups = [&](auto&& pair) { sweep_list<(sizeof(T) == 8), LPP, Nbr>(row, width, n, r, (int)k, gather, pair); };
    auto tail = [&](auto&& pair) { list_tail<LPP, Nbr>(row, width, n, r, (int)k, gather, pair); };
    T gx[3] = {0, 0, 0}, gr = 0, tmp[NQ];
    auto combine = [&]() -> T {
        T sum = T(0);
#pragma unroll
        for (int d = 0; d < DIM; ++d) {
#pragma unroll
            for (int q = 0; q < NQ; ++q) tmp[q] = ax[q][d];
            gx[d] = combine_leaves<LPP>(tmp);
            sum += fabs(gx[d]);
        }
#pragma unroll
        for (int q = 0; q < NQ; ++q) tmp[q] = ar[q];
        gr = combine_leaves<LPP>(tmp);
        return sum + fabs(gr);
    };
    clear();
    if (wave_inside<T, DIM>(K.u, S.H, S.L)) pairs(std::false_type{}, groups);
    else pairs(std::true_type{}, groups);
    pairs(std::true_type{}, tail);
    if (__builtin_expect(!isfinite(combine()), 0) && past_support(sims[psim[opaque(k)]])) {
        const int64_t k2 = opaque(k);
        const PairConst<T> c2 = pair_const(sims[psim[k2]]);
        RenormAdjSelf<T> K2;
        load_self(k2, K2);
        clear();
        walk_again<LPP, Nbr>(nbr + k2 * width, width, nbr_count[k2], r, gather, [&](int q, Nbr& nb) {
            T e[3] = {0, 0, 0};
            const T r2 = r2_exact<T, DIM>(K2.u, nb.a, c2.L, c2.invL, e);
            if (r2 < c2.H2) add(K2, c2.m, c2.invH, c2.hc, nb, e, r2, ax[q], ar[q]);
        });
        combine();
    }
    if (r != 0) return;
    const int o = orig[k];
#pragma unroll
    for (int d = 0; d < DIM; ++d) cot.x[d][o] += c.kGF * gx[d];
    cot.rho[o] += c.kGF * gr;
}

// ---------------------------------------------------------------- particle shifting
//
// dr_i = -beta H^2 sum_j phi_ij V_j grad_i W_ij, phi = 1 + R (W_ij / W(dx))^4, R = 0.2 (the
// delta-plus form; a post-processing step on a state, x <- x + dr).  Same list traversal and
// partial sums as the sweeps; x is updated in original order.
constexpr double kShiftR = 0.2;

template <typename T>
struct ShiftNbr {
    vec4_t<T> a, b;
    __device__ __forceinline__ void keep() { pin(a); }
};

template <typename T, int DIM, int LPP>
__global__ __launch_bounds__(256) void k_shift(int64_t N, int32_t width, const int32_t* __restrict__ nbr,
                                               const int32_t* __restrict__ nbr_count,
                                               const vec4_t<T>* __restrict__ jd0, const int32_t* __restrict__ orig,
                                               const int32_t* __restrict__ psim,
                                               const SimConst<T>* __restrict__ sims, T beta,
                                               StatePtrs<T, DIM> state)
{
    constexpr int NQ = kLeaves / LPP;
    const int64_t t = (int64_t)xcd_remap(blockIdx.x, gridDim.x) * blockDim.x + threadIdx.x;
    const int64_t i = t / LPP;
    const int r = (int)(t - i * LPP);
    if (i >= N) return;
    const SimConst<T>& S = sims[psim[i]];
    const PairConst<T> c = pair_const(S);
    T ui[3] = {0, 0, 0};
    unpack_u<T, DIM>(jd0[i], ui);
    int n = nbr_count[i];
    n = n < width ? n : width;
    const int32_t* row = nbr + i * (int64_t)width;
    T acc[NQ][3];
    auto gather = [&](int j, ShiftNbr<T>& nb) { nb.a = ldo(jd0, (uint32_t)j); };
    auto clear = [&]() {
#pragma unroll
        for (int q = 0; q < NQ; ++q) acc[q][0] = acc[q][1] = acc[q][2] = T(0);
    };
    auto pair = [&](auto within, int q, ShiftNbr<T>& nb) {
        T d[3] = {0, 0, 0};
        const T r2 = r2_exact<T, DIM>(ui, nb.a, c.L, c.invL, d);
        if (decltype(within)::value && !(r2 < c.H2)) return;
        const T tt = kernel_t(r2, c.invH);
        const T qq = fast_sqrt(r2) * c.invH;
        const T t2 = tt * tt;
        const T t4 = t2 * t2;
        const T wr = S.kW * t4 * t2 * (T(1) + qq * (T(6) + qq * T(35.0 / 3.0))) * S.invW0;   // W / W(dx)
        const T w2 = wr * wr;
        const T phi = T(1) + T(kShiftR) * w2 * w2;
        const T f = phi * rec_volume<T, DIM>(nb.a, S.m) * (t4 * (tt * fma(T(-5), tt, T(6))));
#pragma unroll
        for (int k = 0; k < DIM; ++k) acc[q][k] = fma(f, d[k], acc[q][k]);
    };
    auto every = [&](int q, ShiftNbr<T>& nb) { pair(std::false_type{}, q, nb); };
    T sum[3] = {0, 0, 0}, tmp[NQ];
    auto combine = [&]() -> T {
        T mag = T(0);
#pragma unroll
        for (int k = 0; k < DIM; ++k) {
#pragma unroll
            for (int q = 0; q < NQ; ++q) tmp[q] = acc[q][k];
            sum[k] = combine_leaves<LPP>(tmp);
            mag += fabs(sum[k]);
        }
        return mag;
    };
    clear();
    sweep_list<(sizeof(T) == 8), LPP, ShiftNbr<T>>(row, width, n, r, (int)i, gather, every);
    list_tail<LPP, ShiftNbr<T>>(row, width, n, r, (int)i, gather, every);
    if (__builtin_expect(!isfinite(combine()), 0) && past_support(S)) {
        clear();
        walk_again<LPP, ShiftNbr<T>>(row, width, n, r, gather,
                                     [&](int q, ShiftNbr<T>& nb) { pair(std::true_type{}, q, nb); });
        combine();
    }
    if (r != 0) return;
    const int o = orig[i];
    const T cs = -beta * S.H2 * c.kGF;
#pragma unroll
    for (int k = 0; k < DIM; ++k) state.x[k][o] += cs * sum[k];
}

// The position cotangents in sorted order, one record per particle, for k_shift_adj.
template <typename T, int DIM>
__global__ __launch_bounds__(256) void k_pack_xbar(int64_t N, StatePtrs<T, DIM> cot, const int32_t* __restrict__ orig,
                                                   vec4_t<T>* __restrict__ xs)
{
    const int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (k >= N) return;
    const int o = orig[k];
    vec4_t<T> a;
    a.x = cot.x[0][o];
    a.y = cot.x[1][o];
    a.z = (DIM == 3) ? cot.x[2][o] : T(0);
    a.w = T(0);
    xs[k] = a;
}

// Vector-Jacobian product of the shift for cotangents xb of the shifted positions (xs: xb in
// sorted order, one record per particle).  With D(e) = phi Jg + dphi (gF e)(gF e)^T the
// derivative of phi(e) grad W(e), dphi = 4 R (W / W(dx))^3 / W(dx), c = -beta H^2:
//   xbar_k += c sum_j D(e_kj) (V_j xb_k - V_k xb_j)
//   rbar_k += (V_k / rho_k) c sum_j phi gF (e_kj . xb_j)
// added to the cotangents (original order); velocities do not enter.
template <typename T, int DIM, int LPP>
__global__ __launch_bounds__(256) void k_shift_adj(int64_t N, int32_t width, const int32_t* __restrict__ nbr,
                                                   const int32_t* __restrict__ nbr_count,
                                                   const vec4_t<T>* __restrict__ jd0,
                                                   const vec4_t<T>* __restrict__ xs, const T* __restrict__ rho_s,
                                                   const int32_t* __restrict__ orig, const int32_t* __restrict__ psim,
                                                   const SimConst<T>* __restrict__ sims, T beta,
                                                   StatePtrs<T, DIM> cot)
{
    constexpr int NQ = kLeaves / LPP;
    const int64_t t = (int64_t)xcd_remap(blockIdx.x, gridDim.x) * blockDim.x + threadIdx.x;
    const int64_t k = t / LPP;
    const int r = (int)(t - k * LPP);
    if (k >= N) return;
    const SimConst<T>& S = sims[psim[k]];
    const PairConst<T> c = pair_const(S);
    const vec4_t<T> a0 = jd0[k];
    T uk[3] = {0, 0, 0};
    unpack_u<T, DIM>(a0, uk);
    const T Vk = rec_volume<T, DIM>(a0, S.m);
    const vec4_t<T> xk4 = xs[k];
    const T xbk[3] = {xk4.x, xk4.y, xk4.z};
    int n = nbr_count[k];
    n = n < width ? n : width;
    const int32_t* row = nbr + k * (int64_t)width;
    T ax[NQ][3], ar[NQ];
    auto clear = [&]() {
#pragma unroll
        for (int q = 0; q < NQ; ++q) ax[q][0] = ax[q][1] = ax[q][2] = ar[q] = T(0);
    };
    auto gather = [&](int j, ShiftNbr<T>& nb) {
        nb.a = ldo(jd0, (uint32_t)j);
        nb.b = ldo(xs, (uint32_t)j);
    };
    auto pair = [&](auto within, int q, ShiftNbr<T>& nb) {
#pragma clang fp contract(off)
        T e[3] = {0, 0, 0};
        const T r2 = r2_exact<T, DIM>(uk, nb.a, c.L, c.invL, e);
        if (decltype(within)::value && !(r2 < c.H2)) return;
        const T tt = kernel_t(r2, c.invH);
        const T qq = fast_sqrt(r2) * c.invH;
        const T t2 = tt * tt;
        const T t4 = t2 * t2;
        const T gF = t4 * (tt * fma(T(-5), tt, T(6)));   // times kGF at the end
        const T hF = c.hc * t4;
        const T wr = S.kW * t4 * t2 * (T(1) + qq * (T(6) + qq * T(35.0 / 3.0))) * S.invW0;
        const T w2 = wr * wr;
        const T phi = T(1) + T(kShiftR) * w2 * w2;
        const T dphi = T(4.0 * kShiftR) * w2 * wr * S.invW0;
        const T Vj = rec_volume<T, DIM>(nb.a, S.m);
        const T xbj[3] = {nb.b.x, nb.b.y, nb.b.z};
        // z = V_j xb_k - V_k xb_j (zero for the particle itself: no contraction);
        // D z = phi (gF z + hF (e.z) e) + dphi gF^2 (e.z) e
        T z[3], ez = T(0), exj = T(0);
#pragma unroll
        for (int d = 0; d < DIM; ++d) {
            z[d] = Vj * xbk[d] - Vk * xbj[d];
            ez = fma(e[d], z[d], ez);
            exj = fma(e[d], xbj[d], exj);
        }
        const T ce = ez * fma(phi, hF, dphi * (c.kGF * gF) * gF);
        const T pg = phi * gF;
#pragma unroll
        for (int d = 0; d < DIM; ++d) ax[q][d] = fma(pg, z[d], fma(ce, e[d], ax[q][d]));
        ar[q] = fma(pg, exj, ar[q]);
    };
    auto every = [&](int q, ShiftNbr<T>& nb) { pair(std::false_type{}, q, nb); };
    T gx[3] = {0, 0, 0}, gr = 0, tmp[NQ];
    auto combine = [&]() -> T {
        T sum = T(0);
#pragma unroll
        for (int d = 0; d < DIM; ++d) {
#pragma unroll
            for (int q = 0; q < NQ; ++q) tmp[q] = ax[q][d];
            gx[d] = combine_leaves<LPP>(tmp);
            sum += fabs(gx[d]);
        }
#pragma unroll
        for (int q = 0; q < NQ; ++q) tmp[q] = ar[q];
        gr = combine_leaves<LPP>(tmp);
        return sum + fabs(gr);
    };
    clear();
    sweep_list<(sizeof(T) == 8), LPP, ShiftNbr<T>>(row, width, n, r, (int)k, gather, every);
    list_tail<LPP, ShiftNbr<T>>(row, width, n, r, (int)k, gather, every);
    if (__builtin_expect(!isfinite(combine()), 0) && past_support(S)) {
        clear();
        walk_again<LPP, ShiftNbr<T>>(row, width, n, r, gather,
                                     [&](int q, ShiftNbr<T>& nb) { pair(std::true_type{}, q, nb); });
        combine();
    }
    if (r != 0) return;
    const int o = orig[k];
    const T cs = -beta * S.H2 * c.kGF;
#pragma unroll
    for (int d = 0; d < DIM; ++d) cot.x[d][o] += cs * gx[d];
    cot.rho[o] += cs * (Vk / rho_s[k]) * gr;
}

// ---------------------------------------------------------------- neighbour export (CSR, original indices)

__global__ __launch_bounds__(256) void k_export_counts(int64_t N, const int32_t* __restrict__ orig,
                                                       const int32_t* __restrict__ nbr_count, int32_t width,
                                                       int64_t* __restrict__ rowcnt)
{
    int64_t q = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (q >= N) return;
    int c = nbr_count[q];
    rowcnt[orig[q]] = c < width ? c : width;
}

// One wavefront per row: entries mapped to original indices and written in ascending order.
// Up to 64 entries (2D supports) a lane holds one entry and counts the smaller ones, taken from the
// other lanes' registers.  Longer rows (3D) go through a bucket sort in LDS: the bucket is a
// monotone function of the index between the row's smallest and largest, so a row is sorted once
// every bucket is, and an entry's place inside its bucket is a count over the bucket's few members
// (read as aligned quads; cap is a multiple of 4).
// The comparisons per entry fall from the row's length to the bucket's; rows past `cap` entries
// (dense clusters) are ranked against the full row, 64 entries at a time.
// Bound: instruction issue and LDS latency.  3D, 64 000 rows of 257 entries: 107 us against
// 2108 us with every row ranked against itself.
constexpr int kExportCap = 1024;      // longest row sorted in LDS
constexpr int kExportBuckets = 512;
// LDS ints of a row, for rows of at most `cap` entries (a multiple of 4)
constexpr int export_lds_ints(int cap) { return 2 * cap + 8 + kExportBuckets + 4; }

// Orders a wavefront's LDS accesses (the LDS serves one wavefront's accesses in order, so only the
// compiler has to keep them so).
__device__ __forceinline__ void wave_sync()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

constexpr int kExportRows = 4;        // wavefronts, each with a row of its own, per workgroup

__global__ __launch_bounds__(64 * kExportRows) void k_export_rows(int64_t N, int32_t width, const int32_t* __restrict__ orig,
                                                    const int32_t* __restrict__ nbr,
                                                    const int32_t* __restrict__ nbr_count,
                                                    const int64_t* __restrict__ offsets, int32_t* __restrict__ out,
                                                    int cap)
{
    extern __shared__ __align__(16) int32_t export_lds[];
    // cap + 8: the entries by bucket, read as quads
    int32_t* tmp = export_lds + (threadIdx.x >> 6) * export_lds_ints(cap);
    int32_t* row = tmp + cap + 8;
    int32_t* start = row + cap;
    const int64_t q = (int64_t)xcd_remap(blockIdx.x, gridDim.x) * kExportRows + (threadIdx.x >> 6);
    if (q >= N) return;
    const int lane = threadIdx.x & 63;
    int c = nbr_count[q];
    c = __builtin_amdgcn_readfirstlane(c < width ? c : width);
    const int32_t* src = nbr + q * (int64_t)width;
    const int64_t base = offsets[orig[q]];
    if (c <= 64) {
        const int v = lane < c ? orig[src[list_offset(lane, width)]] : 0;
        int rank = 0;
        for (int k = 0; k < c; ++k) rank += (__builtin_amdgcn_readlane(v, k) < v) ? 1 : 0;
        if (lane < c) out[base + rank] = v;
        return;
    }
    if (c <= cap) {
        int lo = INT32_MAX, hi = INT32_MIN;
        for (int m0 = lane; m0 < c; m0 += 256) {   // four entries of a lane in flight; past the row, its last
            int v[4];
#pragma unroll
            for (int j = 0; j < 4; ++j) v[j] = src[list_offset(m0 + 64 * j < c ? m0 + 64 * j : c - 1, width)];
#pragma unroll
            for (int j = 0; j < 4; ++j) v[j] = orig[v[j]];
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                if (m0 + 64 * j < c) row[m0 + 64 * j] = v[j];
                lo = v[j] < lo ? v[j] : lo;
                hi = v[j] > hi ? v[j] : hi;
            }
        }
        for (int b = lane; b < kExportBuckets; b += 64) start[b] = 0;
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) {
            const int l2 = __shfl_xor(lo, o, 64), h2 = __shfl_xor(hi, o, 64);
            lo = l2 < lo ? l2 : lo;
            hi = h2 > hi ? h2 : hi;
        }
        // non-decreasing in v, and at most kExportBuckets - 1 (entries are distinct, so hi > lo)
        const float scale = float(kExportBuckets - 1) / float(hi - lo);
        auto bucket = [&](int v) { return (int)(float(v - lo) * scale); };
        wave_sync();
        // a lane takes `per` consecutive entries, so that the lanes of one atomic reach across the row:
        // neighbouring entries (one cell's particles) mostly share a bucket, and atomics on one
        // address are served one after the other.  per is odd, against bank conflicts.
        const int per = ((c + 63) >> 6) | 1;
        const int first = lane * per, last = first + per < c ? first + per : c;
        for (int m = first; m < last; ++m) atomicAdd(&start[bucket(row[m])], 1);
        wave_sync();
        {
            // bucket counts to bucket ends, in place: eight consecutive buckets a lane
            constexpr int kPer = kExportBuckets / 64;
            int n[kPer], sum = 0;
#pragma unroll
            for (int k = 0; k < kPer; ++k) {
                n[k] = start[kPer * lane + k];
                sum += n[k];
            }
            int end = wave_incl_scan(sum) - sum;
#pragma unroll
            for (int k = 0; k < kPer; ++k) {
                end += n[k];
                start[kPer * lane + k] = end;
            }
            if (lane == 0) start[kExportBuckets] = c;
            if (lane < 8) tmp[c + lane] = INT32_MAX;
        }
        wave_sync();
        // filled from the back, so an end becomes its bucket's start
        for (int m = first; m < last; ++m) {
            const int v = row[m];
            tmp[atomicSub(&start[bucket(v)], 1) - 1] = v;
        }
        wave_sync();
        const int pad = (c + 3) & ~3;   // a quad of INT32_MAX
        for (int m0 = lane; m0 < c; m0 += 256) {
            // aligned quads over the bucket: an entry of an earlier bucket is smaller and counts, one of
            // a later bucket (or the padding) is larger and does not
            int v[4], k[4], e[4], rank[4], more = 0;
#pragma unroll
            for (int j = 0; j < 4; ++j) v[j] = tmp[m0 + 64 * j < c ? m0 + 64 * j : c - 1];
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const int b = bucket(v[j]);
                k[j] = rank[j] = start[b] & ~3;
                e[j] = start[b + 1];
                more |= k[j] < e[j];
            }
            while (more) {
                more = 0;
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    const int4 w = *reinterpret_cast<const int4*>(&tmp[k[j] < e[j] ? k[j] : pad]);
                    rank[j] += (w.x < v[j]) + (w.y < v[j]) + (w.z < v[j]) + (w.w < v[j]);
                    k[j] += 4;
                    more |= k[j] < e[j];
                }
            }
#pragma unroll
            for (int j = 0; j < 4; ++j)
                if (m0 + 64 * j < c) row[rank[j]] = v[j];
        }
        wave_sync();
        for (int m = lane; m < c; m += 64) out[base + m] = row[m];
        return;
    }
    for (int m0 = 0; m0 < c; m0 += 64) {
        const int v = m0 + lane < c ? orig[src[list_offset(m0 + lane, width)]] : 0;
        int rank = 0;
        for (int k0 = 0; k0 < c; k0 += 64) {
            const int w = k0 + lane < c ? orig[src[list_offset(k0 + lane, width)]] : 0;
            const int kn = c - k0 < 64 ? c - k0 : 64;
            for (int k = 0; k < kn; ++k) rank += (__builtin_amdgcn_readlane(w, k) < v) ? 1 : 0;
        }
        if (m0 + lane < c) out[base + rank] = v;
    }
}


// ---------------------------------------------------------------- per-particle support radii
//
// Neighbour search when every particle carries its own support h_i (Sec. 3.2, "Ensuring
// symmetric interactions"; App. B, the search-radius step).  A particle searching with its own
// support would miss partners whose larger support reaches it, so the search radius s_k
// starts at h_k and is raised by an integer atomic maximum on its bit pattern (positive IEEE
// values order like their bits) to h_i for every i that has k as a neighbour under h_i.  Each
// particle then searches with s_i and keeps the pairs with r_ij < max(h_i, h_j), a symmetric
// relation: if h_i >= h_j the pair lies within h_i <= s_i, else i is a neighbour of j under h_j
// and s_i >= h_j.  One thread per particle in sorted order, candidates from the stencil cells
// (the inner 3^dim when the radius fits half the list radius, on cells sized for that half),
// predicates with the arithmetic of the fixed-support search.  Supports must lie in (0, H].

constexpr int kFlagBadSupport = 8;  // a support outside (0, H] (status words of this search only)

// Stencil half-width a particle of search radius rad visits.
template <typename T>
__device__ __forceinline__ int reach_of(const SimConst<T>& S, T rad)
{
    return (S.sub == 2 && rad * rad <= T(0.25) * S.HL2) ? 1 : S.sub;
}

// Cell coordinates of a wrapped position, as the cell assignment computes them.
template <typename T, int DIM>
__device__ __forceinline__ void cell_of_u(const SimConst<T>& S, const T* u, int* cc)
{
    cc[0] = cell_coord(u[0], S.cinv, S.nc);
    cc[1] = cell_coord(u[1], S.cinv, S.nc);
    cc[2] = (DIM == 3) ? cell_coord(u[2], S.cinv, S.nc) : 0;
}

// Calls f(j, r2) for every particle j of the cells within `reach` of cell cc, in the canonical
// order (stencil offset lexicographic in z, y, x, then sorted order inside a cell).
template <typename T, int DIM, typename F>
__device__ __forceinline__ void for_each_candidate(const SimConst<T>& S, const int32_t* __restrict__ blk_rank,
                                                   const int32_t* __restrict__ cell_start,
                                                   const vec4_t<T>* __restrict__ jd0, const int* cc, const T* ui,
                                                   int reach, F&& f)
{
    const int sw = 2 * S.sub + 1;
    const int zr = (DIM == 3) ? reach : 0;
    for (int oz = -zr; oz <= zr; ++oz)
        for (int oy = -reach; oy <= reach; ++oy)
            for (int ox = -reach; ox <= reach; ++ox) {
                const int u = ((DIM == 3 ? (oz + S.sub) * sw : 0) + (oy + S.sub)) * sw + (ox + S.sub);
                const int code = stencil_entry<DIM>(S, blk_rank, cc, u);
                const int id = code & kStencilIdMask;
                T sh[3];
                sh[0] = T(((code >> kStencilIdBits) & 3) - 1) * S.L;
                sh[1] = T(((code >> (kStencilIdBits + 2)) & 3) - 1) * S.L;
                sh[2] = T(((code >> (kStencilIdBits + 4)) & 3) - 1) * S.L;
                const int j1 = cell_start[id + 1];
                for (int j = cell_start[id]; j < j1; ++j) {
                    T uj[3] = {T(0), T(0), T(0)};
                    unpack_u<T, DIM>(jd0[j], uj);
                    f(j, dist2_exact<T, DIM>(ui, uj, sh));
                }
            }
}

// s <- max(s, v) on the bits (v > 0).
__device__ __forceinline__ void raise_to(float* s, float v)
{
    atomicMax(reinterpret_cast<int*>(s), __float_as_int(v));
}
__device__ __forceinline__ void raise_to(double* s, double v)
{
    atomicMax(reinterpret_cast<unsigned long long*>(s), (unsigned long long)__double_as_longlong(v));
}

// Supports into sorted order, search radii initialised to them, supports checked.
template <typename T>
__global__ __launch_bounds__(256) void k_adapt_prepare(int64_t N, const T* __restrict__ h,
                                                       const int32_t* __restrict__ orig,
                                                       const int32_t* __restrict__ psim,
                                                       const SimConst<T>* __restrict__ sims, T* __restrict__ hs,
                                                       T* __restrict__ sr, int32_t* __restrict__ status)
{
    const int64_t q = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (q >= N) return;
    const int s = psim[q];
    T v = h[orig[q]];
    if (!(v > T(0) && v <= sims[s].H)) {
        atomicOr(&status[s], kFlagBadSupport);
        v = sims[s].H;
    }
    hs[q] = v;
    sr[q] = v;
}

// Search radii: every k within h_i of particle i gets s_k >= h_i.
template <typename T, int DIM>
__global__ __launch_bounds__(256) void k_adapt_radius(int64_t N, const vec4_t<T>* __restrict__ jd0,
                                                      const T* __restrict__ hs, T* __restrict__ sr,
                                                      const int32_t* __restrict__ cell_start,
                                                      const int32_t* __restrict__ psim,
                                                      const SimConst<T>* __restrict__ sims,
                                                      const int32_t* __restrict__ blk_rank)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= N) return;
    const SimConst<T>& S = sims[psim[i]];
    T ui[3] = {T(0), T(0), T(0)};
    unpack_u<T, DIM>(jd0[i], ui);
    int cc[3];
    cell_of_u<T, DIM>(S, ui, cc);
    const T hi = hs[i];
    const T hi2 = hi * hi;
    for_each_candidate<T, DIM>(S, blk_rank, cell_start, jd0, cc, ui, reach_of(S, hi), [&](int j, T r2) {
        // only a partner with a smaller support can need its radius raised
        if (r2 < hi2 && hi > hs[j]) raise_to(sr + j, hi);
    });
}

// Lists: the search of radius s_i keeping r_ij < max(h_i, h_j), row-major (width entries per
// row), counts, overflow flagged.
template <typename T, int DIM>
__global__ __launch_bounds__(256) void k_adapt_build(int64_t N, const vec4_t<T>* __restrict__ jd0,
                                                     const T* __restrict__ hs, const T* __restrict__ sr,
                                                     const int32_t* __restrict__ cell_start,
                                                     const int32_t* __restrict__ psim,
                                                     const SimConst<T>* __restrict__ sims,
                                                     const int32_t* __restrict__ blk_rank, int32_t width,
                                                     int32_t* __restrict__ nbr, int32_t* __restrict__ nbr_count,
                                                     int32_t* __restrict__ status)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= N) return;
    const int s = psim[i];
    const SimConst<T>& S = sims[s];
    T ui[3] = {T(0), T(0), T(0)};
    unpack_u<T, DIM>(jd0[i], ui);
    int cc[3];
    cell_of_u<T, DIM>(S, ui, cc);
    const T hi = hs[i];
    int32_t* row = nbr + i * (int64_t)width;
    int c = 0;
    for_each_candidate<T, DIM>(S, blk_rank, cell_start, jd0, cc, ui, reach_of(S, sr[i]), [&](int j, T r2) {
        const T hj = hs[j];
        const T hm = hi > hj ? hi : hj;
        const T hm2 = hm * hm;
        if (r2 < hm2) {
            if (c < width) row[list_offset(c, width)] = j;
            ++c;
        }
    });
    nbr_count[i] = c;
    if (c > width) atomicOr(&status[s], kFlagOverflow);
}

// Sorted-order values back to original order.
template <typename T>
__global__ __launch_bounds__(256) void k_scatter_orig(int64_t N, const T* __restrict__ in,
                                                      const int32_t* __restrict__ orig, T* __restrict__ out)
{
    const int64_t q = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (q < N) out[orig[q]] = in[q];
}

}  // namespace sph
