// kmc_device.hip -- gfx950 kernels of the DCA collision step (arXiv:1310.3437,
// Section 1): bin, scan, cell-sorted copy, partner search, mutual resolve with
// isotropic centre-of-mass scatter, free stream and boundary conditions.
//
// Built with -ffp-contract=off: the only fused multiply-adds are the fma()
// calls written below, which are part of the step's definition.  Every
// floating-point expression that decides a result is written in the
// definition's order so that results are bit-identical to any other
// IEEE-754 binary64 implementation of the same definition.
#include <type_traits>

#include "kmc_internal.h"

namespace kmc {
namespace {

// --------------------------------------------------------------------------
// Definition pieces
// --------------------------------------------------------------------------

// Cell index along one axis: clamp(floor((x - lo) * inv_h), 0, n - 1).
__device__ __forceinline__ int cell1(double x, double lo, double inv_h, int n)
{
    double f = floor((x - lo) * inv_h);
    if (!(f >= 0.0)) return 0;
    if (f >= (double)n) return n - 1;
    return (int)f;
}

// Density-adaptive bins: index of a point on the finest grid (n 2^L cells)
// along one axis, clamp(floor((x - lo) * (inv_h * 2^L)), 0, n 2^L - 1).
// inv_h * 2^L is exact and the power-of-two scaling commutes with the
// rounding of the product, so the point's cell is this index >> L.
__device__ __forceinline__ int fine1(double x, double lo, double inv_h, int n, int L)
{
    const double f = floor((x - lo) * (inv_h * (double)(1 << L)));
    if (!(f >= 0.0)) return 0;
    const double m = (double)n * (double)(1 << L);
    if (f >= m) return (int)(m - 1.0);
    return (int)f;
}

// Split level of a cell holding `count` particles: the smallest l in 0..L
// with count <= T 8^l, else L.
__device__ __forceinline__ uint32_t split_level(uint32_t count, uint32_t T, int L)
{
    for (int l = 0; l < L; ++l)
        if ((uint64_t)count <= ((uint64_t)T << (3 * l))) return (uint32_t)l;
    return (uint32_t)L;
}

// Index of the sub-bin (leaf) a point falls in inside its cell split at
// level lvl: the sub-bin coordinates are bits L-lvl .. L-1 of the finest
// indices, linearised x fastest.
__device__ __forceinline__ uint32_t leaf_code(const BoxDev& B, int L, uint32_t lvl, double x, double y, double z)
{
    const int sh = L - (int)lvl;
    const uint32_t m = (1u << lvl) - 1u;
    const uint32_t sx = ((uint32_t)fine1(x, B.lo[0], B.inv_h[0], B.nc[0], L) >> sh) & m;
    const uint32_t sy = ((uint32_t)fine1(y, B.lo[1], B.inv_h[1], B.nc[1], L) >> sh) & m;
    const uint32_t sz = ((uint32_t)fine1(z, B.lo[2], B.inv_h[2], B.nc[2], L) >> sh) & m;
    return sx + (m + 1u) * (sy + (m + 1u) * sz);
}

// Image of a partner along one axis, from the two cell indices: the
// partner's image is shifted by -L (+L) when it sits in the last (first)
// cell of a periodic axis and the other particle in the first (last).
__device__ __forceinline__ int wrap_of(int ci, int cj, int n, int periodic)
{
    if (!periodic) return 0;
    int d = cj - ci;
    if (d == n - 1) return -1;
    if (d == -(n - 1)) return 1;
    return 0;
}

// Closest-approach quantities of the ordered pair (searcher, candidate):
// b = r.g, g2 = |g|^2, c2 = |r x g|^2 with a fixed fma order.
struct PairQ {
    double b, g2, c2;
};

__device__ __forceinline__ PairQ pair_q(double rx, double ry, double rz,
                                        double gx, double gy, double gz)
{
    PairQ q;
    q.b = fma(rz, gz, fma(ry, gy, rx * gx));
    q.g2 = fma(gz, gz, fma(gy, gy, gx * gx));
    double cx = fma(ry, gz, -(rz * gy));
    double cy = fma(rz, gx, -(rx * gz));
    double cz = fma(rx, gy, -(ry * gx));
    q.c2 = fma(cz, cz, fma(cy, cy, cx * cx));
    return q;
}

// Partner criteria multiplied through by g2 > 0: closest approach within
// [0, dt] (b <= 0, -b <= dt g2) and inside the interaction diameter
// (c2 < D2 g2, i.e. d_min^2 < D2: sigma/pi for one kind of particle, the
// squared sum of the two radii for particles of several kinds).
__device__ __forceinline__ bool accept(const PairQ& q, double D2, double dt)
{
    return (q.g2 > 0.0) & (q.b <= 0.0) & (-q.b <= dt * q.g2) & (q.c2 < D2 * q.g2);
}

// Full 128-bit product of two 64-bit words from four 32x32 partial
// products (schoolbook); each partial product plus a 64-bit addend fits in
// 64 bits, so every step is one 32x32+64 multiply-add and the low word
// reuses the partial products instead of multiplying again.
__device__ __forceinline__ void mul_wide(uint64_t a, uint64_t b, uint64_t& hi, uint64_t& lo)
{
    const uint32_t a0 = (uint32_t)a, a1 = (uint32_t)(a >> 32);
    const uint32_t b0 = (uint32_t)b, b1 = (uint32_t)(b >> 32);
    const uint64_t p00 = (uint64_t)a0 * b0;
    const uint64_t p01 = (uint64_t)a0 * b1 + (p00 >> 32);
    const uint64_t p10 = (uint64_t)a1 * b0 + (uint32_t)p01;
    hi = (uint64_t)a1 * b1 + (p01 >> 32) + (p10 >> 32);
    lo = (p10 << 32) | (uint32_t)p00;
}

// Philox4x64-10 (Salmon, Moraes, Dror, Shaw, SC'11): two 64x64->128
// multiplications per round, Weyl-sequence key schedule.
__device__ __forceinline__ void philox4x64_10(uint64_t c[4], uint64_t k0, uint64_t k1)
{
    const uint64_t m0 = 0xD2E7470EE14C6C93ull, m1 = 0xCA5A826395121157ull;
    const uint64_t w0 = 0x9E3779B97F4A7C15ull, w1 = 0xBB67AE8584CAA73Bull;
#pragma unroll
    for (int r = 0; r < 10; ++r) {
        if (r > 0) { k0 += w0; k1 += w1; }
        uint64_t hi0, lo0, hi1, lo1;
        mul_wide(m0, c[0], hi0, lo0);
        mul_wide(m1, c[2], hi1, lo1);
        uint64_t n0 = hi1 ^ c[1] ^ k0, n2 = hi0 ^ c[3] ^ k1;
        c[0] = n0; c[1] = lo1; c[2] = n2; c[3] = lo0;
    }
}

// Isotropic unit vector (Marsaglia 1972) for the pair whose smaller id is a:
// block k of Philox with key (seed, 0) and counter (k, a, step, 0) offers two
// candidate points (words 0,1 and 2,3) e = 2 (w >> 11) 2^-53 - 1 in [-1, 1);
// the first with 0 < s = e1^2 + e2^2 < 1 gives
// n = (2 e1 sqrt(1-s), 2 e2 sqrt(1-s), 1 - 2s).
__device__ void direction(uint64_t seed, uint64_t step, uint32_t a, double n[3], int dims)
{
    for (uint64_t blk = 0; blk < 32; ++blk) {
        uint64_t w[4] = {blk, (uint64_t)a, step, 0};
        philox4x64_10(w, seed, 0);
#pragma unroll
        for (int t = 0; t < 2; ++t) {
            double e1 = 2.0 * ((double)(w[2 * t] >> 11) * 0x1.0p-53) - 1.0;
            double e2 = 2.0 * ((double)(w[2 * t + 1] >> 11) * 0x1.0p-53) - 1.0;
            if (dims == 2) {
                // planar: (cos 2phi, sin 2phi) of a point uniform in the unit disk
                const double a1 = e1 * e1, a2 = e2 * e2;
                const double s = a1 + a2;
                if (s > 0.0 && s < 1.0) {
                    n[0] = (a1 - a2) / s;
                    n[1] = ((2.0 * e1) * e2) / s;
                    n[2] = 0.0;
                    return;
                }
            } else {
                double s = e1 * e1 + e2 * e2;
                if (s > 0.0 && s < 1.0) {
                    double f = 2.0 * sqrt(1.0 - s);
                    n[0] = e1 * f;
                    n[1] = e2 * f;
                    n[2] = 1.0 - 2.0 * s;
                    return;
                }
            }
        }
    }
    n[0] = dims == 2 ? 1.0 : 0.0;
    n[1] = 0.0;
    n[2] = dims == 2 ? 0.0 : 1.0;
}

// SplitMix64 output of the packed pair (a << 32 | b): the digest term.
__device__ __forceinline__ uint64_t pair_hash(uint32_t a, uint32_t b)
{
    uint64_t z = (((uint64_t)a << 32) | (uint64_t)b) + 0x9E3779B97F4A7C15ull;
    z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
    z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
    return z ^ (z >> 31);
}

// Logical block index for kernels whose neighbouring blocks share data:
// the dispatcher hands consecutive workgroups to the 8 XCDs in turn, each
// with its own L2, so block b is mapped to a contiguous per-XCD range of
// tiles (a bijection for any grid size) and each XCD sweeps one slice of
// the cell-sorted particles.
constexpr uint32_t kXcds = 8;

__device__ __forceinline__ uint32_t xcd_tile(uint32_t b, uint32_t nb)
{
    const uint32_t x = b % kXcds, idx = b / kXcds, q = nb / kXcds, r = nb % kXcds;
    return x * q + (x < r ? x : r) + idx;
}

__device__ __forceinline__ const BoxDev& box_of(const Plan& p, uint32_t i)
{
    return p.boxes[p.boxidx ? p.boxidx[i] : 0u];
}

// Visit the 27-cell neighbourhood of cell (cx, cy, cz) as contiguous ranges
// [s, e) of the cell-sorted arrays: per neighbour row (dy, dz) the cells
// cx-1..cx+1 that exist without wrapping form one range; on a periodic x axis
// a wrapped end cell is a separate range.  f(s, e, wx, wy, wz) receives the
// image selectors of the range.
template <class F>
__device__ __forceinline__ void for_each_range(const BoxDev& B, int cx, int cy, int cz,
                                               const uint32_t* __restrict__ start, F&& f)
{
    const int NX = B.nc[0], NY = B.nc[1], NZ = B.nc[2];
    for (int dz = -1; dz <= 1; ++dz) {
        int nz = cz + dz, wz = 0;
        if (nz < 0) { if (!B.periodic[2]) continue; nz += NZ; wz = -1; }
        else if (nz >= NZ) { if (!B.periodic[2]) continue; nz -= NZ; wz = 1; }
        for (int dy = -1; dy <= 1; ++dy) {
            int ny = cy + dy, wy = 0;
            if (ny < 0) { if (!B.periodic[1]) continue; ny += NY; wy = -1; }
            else if (ny >= NY) { if (!B.periodic[1]) continue; ny -= NY; wy = 1; }
            const uint32_t row = B.coff + (uint32_t)NX * ((uint32_t)ny + (uint32_t)NY * (uint32_t)nz);
            const int x0 = cx - 1, x1 = cx + 1;
            const int m0 = x0 < 0 ? 0 : x0;
            const int m1 = x1 >= NX ? NX - 1 : x1;
            f(start[row + m0], start[row + m1 + 1], 0, wy, wz);
            if (B.periodic[0]) {
                if (x0 < 0) f(start[row + NX - 1], start[row + NX], -1, wy, wz);
                if (x1 >= NX) f(start[row], start[row + 1], 1, wy, wz);
            }
        }
    }
}

// Block-wide sum of two 64-bit values; thread 0 gets the totals.
__device__ __forceinline__ void block_sum2(uint64_t& a, uint64_t& b, uint64_t* lds /*[2*16]*/)
{
    const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6, nw = (blockDim.x + 63) >> 6;
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) {
        a += __shfl_down(a, off, 64);
        b += __shfl_down(b, off, 64);
    }
    if (lane == 0) { lds[wid] = a; lds[16 + wid] = b; }
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int w = 1; w < nw; ++w) { a += lds[w]; b += lds[16 + w]; }
    }
}

// --------------------------------------------------------------------------
// Initialisation and read-back
// --------------------------------------------------------------------------

__global__ void k_init_particles(Plan p, const double* __restrict__ in, const uint8_t* __restrict__ kind)
{
    const uint32_t i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= p.N) return;
    const size_t N = p.N;
    P64 r;
    r.x = in[i];
    r.y = in[N + i];
    r.z = in[2 * N + i];
    r.vx = in[3 * N + i];
    r.vy = in[4 * N + i];
    r.vz = in[5 * N + i];
    p.A[i] = r;
    p.idA[i] = i;
    if (p.spA) {
        // an invalid kind is counted by k_check_kinds (the context is then not
        // created); it is clamped here so that no table read leaves its table
        const uint8_t k = kind[i];
        p.spA[i] = k < (uint8_t)p.nspecies ? k : (uint8_t)(p.nspecies - 1);
    }
    if (p.boxidx) {
        uint32_t lo = 0, hi = p.nboxes - 1;   // last box with poff <= i
        while (lo < hi) {
            uint32_t mid = (lo + hi + 1) >> 1;
            if (p.boxes[mid].poff <= i) lo = mid; else hi = mid - 1;
        }
        p.boxidx[i] = lo;
    }
}

__global__ void k_fill_u32(uint32_t* __restrict__ a, size_t n, uint32_t v)
{
    for (size_t i = blockIdx.x * (size_t)blockDim.x + threadIdx.x; i < n; i += (size_t)gridDim.x * blockDim.x) a[i] = v;
}

__global__ void k_init_ctl(Plan p, unsigned long long step0)
{
    const uint32_t t = threadIdx.x;
    if (t == 0) {
        p.ctl->step = step0;
        p.ctl->steps_done = 0;
        p.ctl->rechecks_total = 0;
        p.ctl->fallbacks_total = 0;
        p.ctl->recheck_count = 0;
        p.ctl->overflow = 0;
        p.ctl->absorbed_total = 0;
        p.ctl->candidates_total = 0;
        p.ctl->scratch = 0;
        p.ctl->tests_init = 0;
    }
    for (uint32_t k = t; k < (uint32_t)kAccLanes; k += blockDim.x) {
        p.acc[k].np = 0;
        p.acc[k].dig = 0;
        p.acc[k].cand = 0;
    }
    for (uint32_t b = t; b < p.nboxes; b += blockDim.x) p.box_v2[b] = 0ull;
}

// Kinds at or beyond the number of kinds, counted into the control block's
// scratch word (kmc_init reads it back).
__global__ void k_check_kinds(Plan p, const uint8_t* __restrict__ kind)
{
    const uint32_t i = blockIdx.x * blockDim.x + threadIdx.x;
    const bool bad = i < p.N && kind[i] >= (uint8_t)p.nspecies;
    const uint64_t m = __ballot(bad);
    if ((threadIdx.x & 63) == 0 && m) atomicAdd(&p.ctl->scratch, (unsigned long long)__popcll(m));
}

__global__ void k_read_partners(Plan p, int32_t* __restrict__ out)
{
    const uint32_t i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= p.N) return;
    const int32_t q = p.partner[i];   // an absorbed particle has none, nor is it anyone's
    out[p.idB[i] & ~kGone] = q >= 0 ? (int32_t)p.idB[q] : -1;
}

__device__ __forceinline__ void store_columns(double* __restrict__ out, size_t N, size_t k, const P64& r)
{
    out[k] = r.x;
    out[N + k] = r.y;
    out[2 * N + k] = r.z;
    out[3 * N + k] = r.vx;
    out[4 * N + k] = r.vy;
    out[5 * N + k] = r.vz;
}

// The state in id order, one launch: every record is read in order and its
// six values go to six random places.
__global__ void k_read_state(Plan p, double* __restrict__ out)
{
    const uint32_t i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= p.N) return;
    store_columns(out, p.N, p.idA[i] & ~kGone, p.A[i]);
}

// The state in id order, two launches: the place of every id (one random
// 4-byte write per particle), then a gather of whole records written out in order.  Both
// are bound by the random accesses: one 48-byte read and one 4-byte write per
// particle instead of the six 8-byte writes of k_read_state, each of which
// costs a memory sector (27.3 -> 6.1 ms at 1e8 particles; the records written
// to their places and transposed from there, without the index, 7.4 to 9 ms).
__global__ void k_state_places(Plan p)
{
    const uint32_t i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= p.N) return;
    p.place[p.idA[i] & ~kGone] = i;
}

__global__ void k_state_gather(Plan p, double* __restrict__ out)
{
    const uint32_t id = blockIdx.x * blockDim.x + threadIdx.x;
    if (id >= p.N) return;
    store_columns(out, p.N, id, p.A[p.place[id]]);
}

// --------------------------------------------------------------------------
// a1: bin + count.  The rank returned by the atomic is the particle's slot
// inside its cell; the order inside a cell never affects a result.
// --------------------------------------------------------------------------

// Cell of particle i at position (x, y, z) and its slot: the state is in
// the previous step's cell order, so neighbouring lanes mostly share a cell
// and each run of equal cells takes its slots with one atomic issued by the
// run's first lane.  Every lane of the wave must call this.
// Global cell of a particle at (x, y, z) in box B; absorbed particles go to
// the box's extra cell after its grid.  On the uniform grid the sorted copy
// recomputes it from the same stored position instead of reading it back;
// with adaptive bins the binning stores it for the leaf count and the copy.
__device__ __forceinline__ uint32_t cell_of(const BoxDev& B, double x, double y, double z, bool gone)
{
    if (gone) return B.coff + (uint32_t)B.nc[0] * (uint32_t)B.nc[1] * (uint32_t)B.nc[2];
    const int cx = cell1(x, B.lo[0], B.inv_h[0], B.nc[0]);
    const int cy = cell1(y, B.lo[1], B.inv_h[1], B.nc[1]);
    const int cz = cell1(z, B.lo[2], B.inv_h[2], B.nc[2]);
    return B.coff + (uint32_t)cx + (uint32_t)B.nc[0] * ((uint32_t)cy + (uint32_t)B.nc[1] * (uint32_t)cz);
}

__device__ __forceinline__ void bin_particle(const Plan& p, uint32_t i, bool valid, const BoxDev& B, double x,
                                             double y, double z, bool gone)
{
    uint32_t c = 0xFFFFFFFFu;
    if (valid) {
        c = cell_of(B, x, y, z, gone);
        if (p.adapt_L > 0) p.cell[i] = c;   // the leaf count reads it back
    }
    const int lane = threadIdx.x & 63;
    const uint64_t live = __ballot(valid);
    if (live == 0) return;
    const uint32_t prev = __shfl_up(c, 1, 64);
    const bool head = valid && (lane == 0 || prev != c);
    const uint64_t H = __ballot(head);
    const uint64_t upto = (2ull << lane) - 1ull;           // lanes 0..lane
    const int my_head = 63 - __clzll((long long)(H & upto));
    const uint64_t above = H & ~upto;
    const int nvalid = __popcll(live);
    const int next = above ? __ffsll((unsigned long long)above) - 1 : nvalid;
    uint32_t base = 0;
    if (head) base = atomicAdd(&p.count[c], (unsigned int)(next - lane));
    base = (uint32_t)__shfl((int)base, my_head, 64);
    if (valid) p.slot[i] = base + (uint32_t)(lane - my_head);
}

// a1 for the state written by kmc_init (later steps bin in k_resolve).
__global__ void k_bin(Plan p)
{
    const uint32_t i = blockIdx.x * blockDim.x + threadIdx.x;
    const bool valid = i < p.N;
    const BoxDev& B = box_of(p, valid ? i : 0u);
    bin_particle(p, i, valid, B, valid ? p.A[i].x : 0.0, valid ? p.A[i].y : 0.0, valid ? p.A[i].z : 0.0, false);
}

// --------------------------------------------------------------------------
// a2: exclusive prefix sum of the cell counts, which also clears the counts
// for the next step: block sums, their scan, down-sweep.  Up to kSumBlocks
// blocks the down-sweep adds up the sums before it itself, and up to
// kOneScanCells cells one block does everything: in a small gas a launch costs
// more than its work (about 4 us each; 2.7e4 cells: three launches 12 us, one
// 7).  Above kNarrowCells the blocks have 1024 threads, so that there are few
// sums (2e7 cells, a million particles: block sums, scan and down-sweep 64 us
// with blocks of 256, 54 with 1024 and no launch between).
// --------------------------------------------------------------------------
constexpr uint32_t kOneScanCells = 32768;

// Start of a step's device-side bookkeeping (recheck list, split cells and
// the FP32 screen's velocity bounds), by one block of the first kernel.
__device__ __forceinline__ void begin_step(const Plan& p)
{
    if (threadIdx.x == 0) {
        p.ctl->recheck_count = 0;
        p.ctl->overflow = 0;
        p.ctl->refined_count = 0;
        p.ctl->pool_used = 0;
    }
    for (uint32_t b = threadIdx.x; b < p.nboxes; b += blockDim.x) p.box_vmax[b] = 0u;
}

__device__ __forceinline__ uint32_t block_exclusive_scan(uint32_t v, uint32_t* lds, uint32_t& total)
{
    const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6, nw = blockDim.x >> 6;
    uint32_t x = v;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
        uint32_t y = __shfl_up(x, off, 64);
        if (lane >= off) x += y;
    }
    if (lane == 63) lds[wid] = x;
    __syncthreads();
    // every wave scans the (at most 16) wave totals for itself
    uint32_t t = lane < nw ? lds[lane] : 0u;
#pragma unroll
    for (int off = 1; off < 16; off <<= 1) {
        const uint32_t y = __shfl_up(t, off, 64);
        if (lane >= off) t += y;
    }
    total = __shfl(t, nw - 1, 64);
    const uint32_t before = __shfl(t, wid > 0 ? wid - 1 : 0, 64);
    __syncthreads();
    return (wid > 0 ? before : 0u) + x - v;
}

// The eight counts of cells base..base+7 (zero beyond the last cell), with
// two 16-byte loads when all eight exist.
__device__ __forceinline__ void load_counts(const Plan& p, uint32_t base, uint32_t v[kScanItems])
{
    static_assert(kScanItems == 8, "two uint4 per thread");
    if (base + kScanItems <= p.C) {
        const uint4* cp = reinterpret_cast<const uint4*>(p.count + base);
        const uint4 a = cp[0], b = cp[1];
        v[0] = a.x; v[1] = a.y; v[2] = a.z; v[3] = a.w;
        v[4] = b.x; v[5] = b.y; v[6] = b.z; v[7] = b.w;
    } else {
#pragma unroll
        for (int k = 0; k < kScanItems; ++k) v[k] = base + k < p.C ? p.count[base + k] : 0u;
    }
}

__global__ __launch_bounds__(1024) void k_scan_reduce(Plan p)
{
    __shared__ uint32_t lds[16];
    const uint32_t base = (blockIdx.x * blockDim.x + threadIdx.x) * kScanItems;
    uint32_t v[kScanItems];
    load_counts(p, base, v);
    uint32_t s = 0;
#pragma unroll
    for (int k = 0; k < kScanItems; ++k) s += v[k];
    uint32_t total;
    block_exclusive_scan(s, lds, total);
    if (threadIdx.x == 0) p.partial[blockIdx.x] = total;
    if (blockIdx.x == 0) begin_step(p);
}

// One block of 1024 threads scans the block sums in place.
__global__ __launch_bounds__(1024) void k_scan_partials(Plan p)
{
    __shared__ uint32_t lds[16];
    uint32_t carry = 0;
    for (uint32_t base = 0; base < p.nblk_scan; base += blockDim.x) {
        const uint32_t k = base + threadIdx.x;
        const uint32_t v = k < p.nblk_scan ? p.partial[k] : 0u;
        uint32_t total;
        const uint32_t e = block_exclusive_scan(v, lds, total);
        if (k < p.nblk_scan) p.partial[k] = carry + e;
        carry += total;
    }
}

// The starts st of the eight cells from base on written, their counts v cleared
// (where there is anything to clear: half of the fours are empty at one
// particle in six cells).
__device__ __forceinline__ void store_starts(const Plan& p, uint32_t base, const uint32_t st[kScanItems],
                                             const uint32_t v[kScanItems])
{
    if (base + kScanItems <= p.C) {
        // 32-byte aligned runs of eight cells (the arrays are 256-byte aligned)
        uint4* sp = reinterpret_cast<uint4*>(p.start + base);
        uint4* cp = reinterpret_cast<uint4*>(p.count + base);
        sp[0] = make_uint4(st[0], st[1], st[2], st[3]);
        sp[1] = make_uint4(st[4], st[5], st[6], st[7]);
        if ((v[0] | v[1] | v[2] | v[3]) != 0u) cp[0] = make_uint4(0u, 0u, 0u, 0u);
        if ((v[4] | v[5] | v[6] | v[7]) != 0u) cp[1] = make_uint4(0u, 0u, 0u, 0u);
    } else {
#pragma unroll
        for (int k = 0; k < kScanItems; ++k) {
            const uint32_t c = base + k;
            if (c < p.C) {
                p.start[c] = st[k];
                p.count[c] = 0u;
            }
        }
    }
}

// The whole scan in one block: four tiles of eight cells per thread, all
// loaded at once; the 64 wave totals are scanned by one wave.
__global__ __launch_bounds__(1024) void k_scan_one(Plan p)
{
    constexpr uint32_t kTiles = kOneScanCells / (1024u * kScanItems);
    static_assert(kTiles * 16u == 64u, "one wave total per lane");
    __shared__ uint32_t wt[64];
    const uint32_t lane = threadIdx.x & 63u, wid = threadIdx.x >> 6;
    uint32_t v[kTiles][kScanItems], x[kTiles], sum[kTiles];
#pragma unroll
    for (uint32_t t = 0; t < kTiles; ++t) load_counts(p, (t * 1024u + threadIdx.x) * kScanItems, v[t]);
#pragma unroll
    for (uint32_t t = 0; t < kTiles; ++t) {
        sum[t] = 0;
#pragma unroll
        for (int k = 0; k < kScanItems; ++k) sum[t] += v[t][k];
        x[t] = sum[t];
#pragma unroll
        for (int off = 1; off < 64; off <<= 1) {
            const uint32_t y = __shfl_up(x[t], off, 64);
            if (lane >= (uint32_t)off) x[t] += y;
        }
        if (lane == 63u) wt[t * 16u + wid] = x[t];
    }
    __syncthreads();
    if (wid == 0) {
        const uint32_t w = wt[lane];
        uint32_t e = w;
#pragma unroll
        for (int off = 1; off < 64; off <<= 1) {
            const uint32_t y = __shfl_up(e, off, 64);
            if (lane >= (uint32_t)off) e += y;
        }
        wt[lane] = e - w;
    }
    __syncthreads();
#pragma unroll
    for (uint32_t t = 0; t < kTiles; ++t) {
        uint32_t run = wt[t * 16u + wid] + x[t] - sum[t];
        uint32_t st[kScanItems];
#pragma unroll
        for (int k = 0; k < kScanItems; ++k) {
            st[k] = run;
            run += v[t][k];
        }
        store_starts(p, (t * 1024u + threadIdx.x) * kScanItems, st, v[t]);
    }
    if (threadIdx.x == 0) p.start[p.C] = p.N;
    begin_step(p);
}

// SUMS: the block sums are as k_scan_reduce left them (else scanned).
template <bool SUMS>
__global__ __launch_bounds__(1024) void k_scan_down(Plan p)
{
    __shared__ uint32_t lds[16];
    uint32_t before = 0;
    if (SUMS) {
        uint32_t a = 0;
        for (uint32_t k = threadIdx.x; k < blockIdx.x; k += blockDim.x) a += p.partial[k];
        block_exclusive_scan(a, lds, before);
    } else {
        before = p.partial[blockIdx.x];
    }
    const uint32_t base = (blockIdx.x * blockDim.x + threadIdx.x) * kScanItems;
    uint32_t v[kScanItems];
    load_counts(p, base, v);
    uint32_t s = 0;
#pragma unroll
    for (int k = 0; k < kScanItems; ++k) s += v[k];
    uint32_t total;
    uint32_t run = block_exclusive_scan(s, lds, total) + before;
    uint32_t st[kScanItems];
#pragma unroll
    for (int k = 0; k < kScanItems; ++k) {
        st[k] = run;
        run += v[k];
    }
    store_starts(p, base, st, v);
    if (blockIdx.x == 0 && threadIdx.x == 0) p.start[p.C] = p.N;
    if (p.adapt_L > 0) {
        // adaptive bins: this step's split level of every cell from its count;
        // split cells are listed and claim their leaf tables (one pair of
        // atomics per block, on two counters that every block shares: the
        // block's split cells take consecutive list entries and pool ranges,
        // in thread order)
        uint64_t lv = 0;
        uint32_t nsplit = 0, need = 0;
#pragma unroll
        for (int k = 0; k < kScanItems; ++k) {
            const uint32_t c = base + k;
            if (c < p.C) {
                const uint32_t l = split_level(v[k], p.adapt_T, p.adapt_L);
                lv |= (uint64_t)l << (8 * k);
                if (l) {
                    nsplit += 1u;
                    need += (1u << (3 * l)) + 1u;
                }
            }
        }
        const int lane = threadIdx.x & 63;
        uint32_t xs = nsplit, xn = need;
#pragma unroll
        for (int off = 1; off < 64; off <<= 1) {
            const uint32_t ys = __shfl_up(xs, off, 64), yn = __shfl_up(xn, off, 64);
            if (lane >= off) {
                xs += ys;
                xn += yn;
            }
        }
        __shared__ uint32_t wsum[2][16];
        const int wid = threadIdx.x >> 6, nw = (int)(blockDim.x >> 6);
        if (lane == 63) {
            wsum[0][wid] = xs;
            wsum[1][wid] = xn;
        }
        __syncthreads();
        if (threadIdx.x == 0) {
            uint32_t ts = 0, tn = 0;
            for (int w = 0; w < nw; ++w) {
                ts += wsum[0][w];
                tn += wsum[1][w];
            }
            uint32_t bs = 0, bn = 0;
            if (ts) {
                bs = atomicAdd(&p.ctl->refined_count, ts);
                bn = atomicAdd(&p.ctl->pool_used, tn);
            }
            for (int w = 0; w < nw; ++w) {   // each wave's first entry and pool offset
                const uint32_t a = wsum[0][w], b = wsum[1][w];
                wsum[0][w] = bs;
                wsum[1][w] = bn;
                bs += a;
                bn += b;
            }
        }
        __syncthreads();
        uint32_t rs = wsum[0][wid] + xs - nsplit;
        uint32_t rn = wsum[1][wid] + xn - need;
#pragma unroll
        for (int k = 0; k < kScanItems; ++k) {
            const uint32_t l = (uint32_t)(lv >> (8 * k)) & 0xFFu;
            if (l) {
                const uint32_t c = base + k;
                p.refined[rs++] = c;
                p.pool_base[c] = rn;
                rn += (1u << (3 * l)) + 1u;
            }
        }
        if (base + kScanItems <= p.C) {
            *reinterpret_cast<uint64_t*>(p.level + base) = lv;
            *reinterpret_cast<uint64_t*>(p.mixed + base) = 0ull;
        } else {
            for (int k = 0; k < kScanItems; ++k)
                if (base + k < p.C) {
                    p.level[base + k] = (uint8_t)(lv >> (8 * k));
                    p.mixed[base + k] = 0;
                }
        }
    }
}

// Box of a global cell (the boxes' cells are consecutive, in box order).
__device__ __forceinline__ uint32_t box_of_cell(const Plan& p, uint32_t c)
{
    uint32_t lo = 0, hi = p.nboxes - 1;
    while (lo < hi) {
        const uint32_t mid = (lo + hi + 1) >> 1;
        if (p.boxes[mid].coff <= c) lo = mid; else hi = mid - 1;
    }
    return lo;
}

// Adaptive bins, per split cell (one wave each): clear its leaf counts and
// mark it and its 26 neighbours as cells whose particles' neighbourhoods
// are not the plain 27 cells.
__global__ __launch_bounds__(64) void k_refined_prep(Plan p)
{
    const uint32_t n = p.ctl->refined_count;
    const uint32_t lane = threadIdx.x;
    for (uint32_t k = blockIdx.x; k < n; k += gridDim.x) {
        const uint32_t c = p.refined[k];
        const uint32_t m = 1u << (3u * p.level[c]);
        const uint32_t pb = p.pool_base[c];
        for (uint32_t t = lane; t < m; t += 64u) p.pool[pb + t] = 0u;
        if (lane < 27u) {
            const BoxDev& B = p.boxes[box_of_cell(p, c)];
            const uint32_t loc = c - B.coff, NX = (uint32_t)B.nc[0], NY = (uint32_t)B.nc[1];
            int q[3] = {(int)(loc % NX), (int)((loc / NX) % NY), (int)(loc / (NX * NY))};
            const int d[3] = {(int)(lane % 3u) - 1, (int)((lane / 3u) % 3u) - 1, (int)(lane / 9u) - 1};
            bool ok = true;
#pragma unroll
            for (int a = 0; a < 3; ++a) {
                q[a] += d[a];
                if (q[a] < 0) { if (B.periodic[a]) q[a] += B.nc[a]; else ok = false; }
                else if (q[a] >= B.nc[a]) { if (B.periodic[a]) q[a] -= B.nc[a]; else ok = false; }
            }
            if (ok) p.mixed[B.coff + (uint32_t)q[0] + NX * ((uint32_t)q[1] + NY * (uint32_t)q[2])] = 1;
        }
    }
}

// Adaptive bins: each particle of a split cell counts itself into its leaf;
// the returned value is its rank in the leaf.  The state is in the previous
// step's leaf order, so neighbouring lanes mostly share a leaf: each run of
// equal leaves takes its ranks with one atomic issued by the run's first lane
// (as the binning does for cells).  Every lane of the wave takes part.
__global__ void k_leaf_count(Plan p)
{
    const uint32_t i = blockIdx.x * blockDim.x + threadIdx.x;
    const uint32_t kNone = 0xFFFFFFFFu;
    uint32_t key = kNone;   // the particle's leaf counter in the pool (none: its cell is not split)
    if (i < p.N) {
        const uint32_t c = p.cell[i];
        const uint32_t lvl = p.level[c];
        if (lvl != 0u) {
            key = p.pool_base[c] + leaf_code(box_of(p, i), p.adapt_L, lvl, p.A[i].x, p.A[i].y, p.A[i].z);
        }
    }
    const int lane = threadIdx.x & 63;
    const bool counted = key != kNone;
    const uint32_t prev = __shfl_up(key, 1, 64);
    const bool cont = counted && lane > 0 && prev == key;   // same leaf as the lane before
    const uint64_t H = __ballot(counted && !cont);          // first lanes of runs
    const uint64_t E = __ballot(!cont);                     // lanes that do not continue a run
    const uint64_t upto = (2ull << lane) - 1ull;            // lanes 0..lane
    const uint64_t after = E & ~upto;
    const int next = after ? __ffsll((unsigned long long)after) - 1 : 64;
    uint32_t base = 0;
    if (counted && !cont) base = atomicAdd(&p.pool[key], (unsigned int)(next - lane));
    const int my_head = counted ? 63 - __clzll((long long)(H & upto)) : lane;
    base = (uint32_t)__shfl((int)base, my_head, 64);
    if (counted) p.leaf_slot[i] = base + (uint32_t)(lane - my_head);
}

// Adaptive bins, per split cell (one wave each): the exclusive prefix of its
// leaf counts in place (leaf starts relative to the cell's start), then the
// cell's count after the last.
__global__ __launch_bounds__(64) void k_leaf_scan(Plan p)
{
    const uint32_t n = p.ctl->refined_count;
    const int lane = threadIdx.x;
    for (uint32_t k = blockIdx.x; k < n; k += gridDim.x) {
        const uint32_t c = p.refined[k];
        const uint32_t m = 1u << (3u * p.level[c]);
        uint32_t* t = p.pool + p.pool_base[c];
        const uint32_t per = m > 64u ? m / 64u : 1u;    // entries per lane (m is 8, 64 or 512)
        const uint32_t b0 = (uint32_t)lane * per;
        uint32_t v[8];
        uint32_t sum = 0;
#pragma unroll
        for (uint32_t e = 0; e < 8u; ++e) {
            v[e] = (e < per && b0 + e < m) ? t[b0 + e] : 0u;
            sum += v[e];
        }
        uint32_t x = sum;
#pragma unroll
        for (int off = 1; off < 64; off <<= 1) {
            const uint32_t y = __shfl_up(x, off, 64);
            if (lane >= off) x += y;
        }
        uint32_t run = x - sum;
#pragma unroll
        for (uint32_t e = 0; e < 8u; ++e) {
            if (e < per && b0 + e < m) t[b0 + e] = run;
            run += v[e];
        }
        if (lane == 63) t[m] = x;
    }
}

// --------------------------------------------------------------------------
// a3: cell-sorted copy of the state as 48-byte records (ids and kinds beside
// them); for the FP32 screen also the per-block bound on |fl32(v_k)| from
// which the screen's error bounds per box are made.
// --------------------------------------------------------------------------

// The screen's error bounds take every particle to lie inside the cell it is
// binned in (up to a slack of 1e-9 of a cell edge).  A particle outside its
// box's grid (placed there, or moved more than a box length in one step) is
// binned in an end cell; the step's partners then come from the whole-step
// FP64 search instead.  Rounding-level excursions (a sphere's mirror image
// just past a face of a grid that fits it exactly) stay within the slack and
// are ignored.
__device__ __forceinline__ bool outside_grid(const BoxDev& B, const P64& r)
{
    bool out = !(r.x >= B.lo[0] && r.x <= B.hi[0] && r.y >= B.lo[1] && r.y <= B.hi[1] && r.z >= B.lo[2] &&
                 r.z <= B.hi[2]);
    if (out) {
        const double t0 = 1e-11 * B.h[0], t1 = 1e-11 * B.h[1], t2 = 1e-11 * B.h[2];
        out = !(r.x >= B.lo[0] - t0 && r.x <= B.hi[0] + t0 && r.y >= B.lo[1] - t1 && r.y <= B.hi[1] + t1 &&
                r.z >= B.lo[2] - t2 && r.z <= B.hi[2] + t2);
    }
    return out;
}

template <bool F32>
__global__ void k_scatter(Plan p)
{
    const uint32_t i = blockIdx.x * blockDim.x + threadIdx.x;
    const bool valid = i < p.N;
    float vm = 0.f;
    bool outside = false;
    double vx = 0.0, vy = 0.0, vz = 0.0;
    // the particle's box; one box (no per-particle index): the same for the
    // whole grid, read through scalar loads
    auto body = [&](const BoxDev& B) {
        const uint32_t id = p.idA[i];
        const P64 r = p.A[i];
        const uint32_t c = p.adapt_L > 0 ? p.cell[i] : cell_of(B, r.x, r.y, r.z, (id & kGone) != 0u);
        uint32_t d = p.start[c] + p.slot[i];
        if (p.adapt_L > 0) {
            // adaptive bins: leaf-sorted inside a split cell
            const uint32_t lvl = p.level[c];
            if (lvl) {
                const uint32_t code = leaf_code(B, p.adapt_L, lvl, r.x, r.y, r.z);
                d = p.start[c] + p.pool[p.pool_base[c] + code] + p.leaf_slot[i];
            }
        }
        vx = r.vx;
        vy = r.vy;
        vz = r.vz;
        p.B[d] = r;
        p.idB[d] = id;
        if (p.spA) p.spB[d] = p.spA[i];
        if (id & kGone) vx = vy = vz = 0.0;   // not in the gas: no part in the adaptive step
        if (F32) {
            vm = fmaxf(fabsf((float)r.vx), fmaxf(fabsf((float)r.vy), fabsf((float)r.vz)));
            // (a box's largest speed is 0 only where every particle rests)
            if (vm == 0.f && ((r.vx != 0.0) | (r.vy != 0.0) | (r.vz != 0.0))) vm = 0x1p-126f;
            if (!(id & kGone)) {
                outside = outside_grid(B, r);
            }
        }
    };
    if (valid) {
        if (p.boxidx) body(p.boxes[p.boxidx[i]]);
        else body(p.boxes[0]);
    }
    __shared__ float wmax[16];
    __shared__ unsigned long long wv2[16];
    if (F32) {
        if (__ballot(outside) && (threadIdx.x & 63) == 0) atomicOr(&p.ctl->overflow, 1u);
        // per-block maximum of |fl32(v_k)|; fold_partials takes those of each box
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) vm = fmaxf(vm, __shfl_xor(vm, off, 64));
        if ((threadIdx.x & 63) == 0) wmax[threadIdx.x >> 6] = vm;
    }
    if (p.dt_rule == KMC_DT_ADAPTIVE) {
        // adaptive time step: max |v|^2 per box.  Non-negative doubles order
        // like their bit patterns, so the maximum is exact in any order.  The
        // block folds its particles that share the box of its first particle
        // (fold_partials reads the partial); any others go to their box directly.
        const uint32_t first = blockIdx.x * blockDim.x;
        const uint32_t b0 = p.boxidx ? p.boxidx[first] : 0u;
        unsigned long long q = 0ull;
        if (valid) {
            const double v2 = fma(vz, vz, fma(vy, vy, vx * vx));
            const unsigned long long bits = (unsigned long long)__double_as_longlong(v2);
            const uint32_t bi = p.boxidx ? p.boxidx[i] : 0u;
            if (bi == b0) q = bits;
            else atomicMax(&p.box_v2[bi], bits);
        }
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) {
            const unsigned long long o = __shfl_xor(q, off, 64);
            q = o > q ? o : q;
        }
        if ((threadIdx.x & 63) == 0) wv2[threadIdx.x >> 6] = q;
    }
    if (F32 || p.dt_rule == KMC_DT_ADAPTIVE) {
        __syncthreads();
        if (threadIdx.x == 0) {
            const int nw = (int)(blockDim.x >> 6);
            if (F32) {
                float m = 0.f;
                for (int w = 0; w < nw; ++w) m = fmaxf(m, wmax[w]);
                p.vmax_part[blockIdx.x] = m;
            }
            if (p.dt_rule == KMC_DT_ADAPTIVE) {
                unsigned long long m = 0ull;
                for (int w = 0; w < nw; ++w) m = wv2[w] > m ? wv2[w] : m;
                p.v2_part[blockIdx.x] = m;
            }
        }
    }
}

// The adaptive rule's step from the bits of max |v|^2.
__device__ __forceinline__ double adaptive_dt(const Plan& p, const BoxDev& B, unsigned long long v2_bits)
{
    const double v2 = __longlong_as_double((long long)v2_bits);
    double dt = B.dt_cap;
    if (v2 > 0.0) {
        const double a = (p.dt_factor * B.dx) / sqrt(v2);
        if (a < dt) dt = a;
    }
    return dt;
}

// Maxima of a box's scatter blocks k = first + part, first + part + stride, ...
// (a block of 256 threads): |v|^2 over the blocks whose first particle lies in
// the box, and |fl32(v_k)| over all blocks that touch it.  Thread 0 gets them.
__device__ __forceinline__ void fold_partials(const Plan& p, const BoxDev& B, uint32_t part, uint32_t stride,
                                              unsigned long long& v2, float& vm)
{
    __shared__ unsigned long long r2[4];
    __shared__ float rv[4];
    v2 = 0ull;
    vm = 0.f;
    if (B.n > 0) {
        const uint32_t blk = (uint32_t)p.block;
        const uint32_t first = B.poff / blk, last = (B.poff + B.n - 1) / blk, own = (B.poff + blk - 1) / blk;
        for (uint32_t k = first + part; k <= last; k += stride) {
            if (p.precision == KMC_FP32_SCREEN) vm = fmaxf(vm, p.vmax_part[k]);
            if (p.dt_rule == KMC_DT_ADAPTIVE && k >= own) {
                const unsigned long long v = p.v2_part[k];
                v2 = v > v2 ? v : v2;
            }
        }
    }
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) {
        const unsigned long long o = __shfl_xor(v2, off, 64);
        v2 = o > v2 ? o : v2;
        vm = fmaxf(vm, __shfl_xor(vm, off, 64));
    }
    if ((threadIdx.x & 63) == 0) {
        r2[threadIdx.x >> 6] = v2;
        rv[threadIdx.x >> 6] = vm;
    }
    __syncthreads();
    if (threadIdx.x == 0)
        for (int w = 1; w < 4; ++w) {
            v2 = r2[w] > v2 ? r2[w] : v2;
            vm = fmaxf(vm, rv[w]);
        }
}

// Boxes of many scatter blocks: kVmaxSplit blocks per box fold the partials
// first, one atomic each (non-negative floats order like their bit patterns).
// One block alone took 62 us for the 3.9e4 partials of 1e7 particles.
constexpr uint32_t kVmaxSplit = 32;
constexpr uint32_t kFoldAlone = 2048;   // scatter blocks of a step that need no help

__global__ __launch_bounds__(256) void k_fold_partials(Plan p)
{
    const uint32_t b = blockIdx.x / kVmaxSplit, part = blockIdx.x % kVmaxSplit;
    unsigned long long v2;
    float vm;
    fold_partials(p, p.boxes[b], part * blockDim.x + threadIdx.x, kVmaxSplit * blockDim.x, v2, vm);
    if (threadIdx.x == 0) {
        if (vm > 0.f) atomicMax(&p.box_vmax[b], __float_as_uint(vm));
        if (v2) atomicMax(&p.box_v2[b], v2);
    }
}

// --------------------------------------------------------------------------
// a4: DCA partner search.
//
// The pair quantities are symmetric under exchange of the two particles
// (r, g and r x g change sign, b, g2, c2 do not), so every unordered pair is
// tested once, from the particle whose cell comes first in a half
// neighbourhood: its own row from the particle onwards through cell cx+1,
// the row y+1 (cells cx-1..cx+1) and the three rows z+1 (y-1..y+1).  A lane
// keeps the pairs that pass; at the end of the wave it decides them exactly
// in FP64, writes the best of them (its forward best) and posts each
// acceptable pair, with its key, to the other particle's candidate list.  A
// per-particle finish pass then takes the (key, id) minimum of the forward
// best and the list.
//
// One wave (= one block of 64 threads) takes 64 consecutive cell-sorted
// particles, one per lane.  Lanes whose particles share a cell row form a
// group; for each of the five half-neighbourhood rows the group's window of
// cells is a contiguous range of the sorted arrays, which the wave stages
// into LDS in chunks with coalesced loads.  Each lane then tests its own
// sub-range of the window from LDS.
// --------------------------------------------------------------------------

// Row of sorted particle i's kind in the kind-pair tables (kMaxKinds * its
// kind; 0 for one kind of particle).
__device__ __forceinline__ uint32_t kind_row(const Plan& p, uint32_t i)
{
    return p.nspecies ? (uint32_t)p.spB[i] * (uint32_t)kMaxKinds : 0u;
}

// Squared interaction diameter of the pair of sorted particles (i, j): the
// box's D2 for one kind of particle, else (radius_s + radius_t)^2 of their
// kinds.
__device__ __forceinline__ double pair_D2(const Plan& p, const BoxDev& B, uint32_t row_i, uint32_t j)
{
    return p.nspecies ? p.sp_D2[row_i + p.spB[j]] : B.D2;
}

// Relative position of candidate j seen from i in FP64 with the image fixed
// by the two cells, exactly as in the search.
__device__ __forceinline__ void rel64(const BoxDev& B, const P64& me, const P64& q, double r[3])
{
    const double xi[3] = {me.x, me.y, me.z}, xj[3] = {q.x, q.y, q.z};
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        const int ci = cell1(xi[k], B.lo[k], B.inv_h[k], B.nc[k]);
        const int cj = cell1(xj[k], B.lo[k], B.inv_h[k], B.nc[k]);
        const int w = wrap_of(ci, cj, B.nc[k], B.periodic[k]);
        r[k] = xj[k] - xi[k];
        if (w != 0) r[k] = r[k] + (double)w * B.L[k];
    }
}

// Candidate lists: per particle a count and up to kSlots entries (sorted
// index of the other particle and the pair's FP64 key c2/g2, which is the
// same from both sides, or +inf for a pair the FP32 screen kept and the exact
// test rejected); entry k of particle i lives at [k * N + i].
__device__ __forceinline__ void post_candidate(const Plan& p, uint32_t i, uint32_t j, double key)
{
    const uint32_t k = atomicAdd(&p.sl_cnt[i], 1u);
    if (k < (uint32_t)kSlots) {
        SlotEntry e;
        e.key = key;
        e.j = j;
        e.pad_ = 0u;
        p.sl[(size_t)k * p.N + i] = e;
    }
}

// The definition's exact FP64 decision for the pair (i, j) seen from i (the
// image from the two cells), and its key when acceptable.
__device__ __forceinline__ bool exact_key(const Plan& p, const BoxDev& B, uint32_t i, const P64& me, uint32_t j,
                                          double& key)
{
    const P64 q = p.B[j];
    double r[3];
    rel64(B, me, q, r);
    const PairQ pq = pair_q(r[0], r[1], r[2], q.vx - me.vx, q.vy - me.vy, q.vz - me.vz);
    if (!accept(pq, pair_D2(p, B, kind_row(p, i), j), B.dt)) return false;
    key = pq.c2 / pq.g2;
    return true;
}

// Pairs a lane found, kept until the end of the wave's search (the sorted
// indices in LDS, the image shifts in a register: a global atomic or a
// division inside the search loop would stall the whole wave).  A lane that
// finds more than kReg appends the excess to the wave's list of extra pairs
// in LDS, which the wave decides and posts together at its end.  When that
// list is full, both particles of a further pair are marked for the full FP64
// re-search.  (Marking a lane's whole window instead made re-searches of whole
// clusters: 1.8e5 particles in four clusters 8.8 ms a step against 4.0.)
// In a Maxwellian gas at three particles per cell (about three acceptable
// partners each) 1.4% of the lanes find more than four; when each of these
// pairs took an atomic on one step-wide counter the search waited on it
// (3e6 particles, FP64: 1320 us, now 420; eight slots per lane instead of the
// wave's list: 437 us, but 8.57 ms against 8.27 on the 1e8 sphere, whose
// registers they take).
constexpr int kReg = 4;
constexpr uint32_t kExtra = 96;
constexpr uint32_t kMarked = 16;   // list count added by a mark (> kSlots)

struct Extra {
    uint32_t n;             // pairs offered (those beyond kExtra were lost)
    uint32_t j[kExtra];     // sorted index of the partner
    uint8_t lane[kExtra];   // the lane that found the pair
};

__device__ __forceinline__ uint32_t wcode(int wx, int wy, int wz)
{
    return (uint32_t)(wx + 1) | ((uint32_t)(wy + 1) << 2) | ((uint32_t)(wz + 1) << 4);
}
constexpr uint32_t kNoImage = 0x15u;   // wcode(0, 0, 0)

// The candidates of a row as a sequence f: their place in the sorted order and
// their image.  Row is the usual one, f the place itself.
struct Row {
    int wx, wy, wz;
    __device__ __forceinline__ uint32_t at(uint32_t f, int& x) const
    {
        x = wx;
        return f;
    }
    __device__ __forceinline__ uint32_t at(uint32_t f, uint32_t& code) const
    {
        code = wcode(wx, wy, wz);
        return f;
    }
};

// A row with the wrapped end cells of a periodic x axis: first the nL
// candidates of the one on the left (sorted from sL on), then the nM of the row
// itself (from gs on), then those of the one on the right (from sR on).
struct WrappedRow {
    uint32_t gs, nM, nL, sL, sR;
    int wy, wz;
    __device__ __forceinline__ uint32_t at(uint32_t f, int& x) const
    {
        const bool l = f < nL, r = f >= nL + nM;
        x = l ? -1 : r ? 1 : 0;
        return f + (l ? sL : r ? sR - nL - nM : gs - nL);
    }
    __device__ __forceinline__ uint32_t at(uint32_t f, uint32_t& code) const
    {
        int x;
        const uint32_t j = at(f, x);
        code = wcode(x, wy, wz);
        return j;
    }
};

struct Found {
    Extra* extra; // the wave's extra pairs in LDS
    uint32_t* sj; // this lane's kept indices in LDS: pair k at sj[64 k] (one store per pair
                  // instead of a select over register slots)
    uint32_t w;   // image shift of pair k in bits 6k..6k+5: (wx+1) | (wy+1) << 2 | (wz+1) << 4;
                  // bit 31: the lane lost a pair
    int n;
    uint32_t* lists;   // lengths of the candidate lists
    __device__ __forceinline__ void clear(Extra* e, uint32_t* slots, uint32_t* l)
    {
        extra = e;
        sj = slots;
        lists = l;
        n = 0;
        w = kNoImage * 0x41041u;   // no image in every slot
    }
    template <class M>
    __device__ __forceinline__ void keep(uint32_t f, const M& m)
    {
        uint32_t code;
        sj[64 * n] = m.at(f, code);
        if (code != kNoImage) w ^= (code ^ kNoImage) << (6 * n);
        ++n;
    }
    // Consecutive candidates f and f + 1, of which at least one is kept (the
    // usual case, one of them with slots to spare, has no branches inside).
    template <class M>
    __device__ __forceinline__ void add2(bool k0, bool k1, uint32_t f, const M& m)
    {
        if (n + 1 < kReg) {
            keep(k0 ? f : f + 1u, m);
            if (k0 & k1) keep(f + 1u, m);
        } else {
            if (k0) add(f, m);
            if (k1) add(f + 1u, m);
        }
    }
    template <class M>
    __device__ __forceinline__ void add(uint32_t f, const M& m)
    {
        if (__builtin_expect(n < kReg, 1)) {
            keep(f, m);
            return;
        }
        const uint32_t t = atomicAdd(&extra->n, 1u);
        uint32_t code;   // (the exact decision finds the image from the cells)
        const uint32_t j = m.at(f, code);
        if (__builtin_expect(t < kExtra, 1)) {
            extra->j[t] = j;
            extra->lane[t] = (uint8_t)threadIdx.x;
        } else {
            uint32_t k = j;
            asm("" : "+v"(k));   // (keeps the address out of the pair loop)
            w |= 0x80000000u;
            (void)atomicAdd(&lists[k], kMarked);
        }
    }
    // Decide the kept pairs exactly in FP64 (the FP32 screen keeps pairs it
    // could not reject), write i's best among them (its forward best) and
    // post each kept pair to the other particle's list (key +inf when the
    // exact test rejects it).  The image shift is the one the search used
    // (that of the two cells).  All lanes take the same path: list slots
    // claimed, records loaded, the arithmetic, then the list entries
    // written.  Returns the number of pairs examined (statistics).
    // BATCH records are loaded at a time; SKIP: no loads for empty slots
    // (otherwise branch-free, loading the own record for them) -- measured
    // per precision
    // K: particles of several kinds (the pair's D2 from the kind table).
    template <int BATCH, bool SKIP, bool K>
    __device__ __forceinline__ uint32_t flush(const Plan& p, uint32_t i, const P64& me, const BoxDev& B)
    {
        const uint32_t row = K ? kind_row(p, i) : 0u;
        uint32_t j[kReg];
#pragma unroll
        for (int k = 0; k < kReg; ++k) j[k] = k < n ? sj[64 * k] : 0u;
        // list slots of the kept pairs claimed first: the atomics are in
        // flight while the records load and the pairs are decided (a pair the
        // FP64 test then rejects leaves an entry with key +inf, which never
        // wins in the finish)
        uint32_t slot[kReg];
#pragma unroll
        for (int k = 0; k < kReg; ++k) slot[k] = k < n ? atomicAdd(&p.sl_cnt[j[k]], 1u) : (uint32_t)kSlots;
        double key[kReg];
        bool acc[kReg];
#pragma unroll
        for (int k = 0; k < kReg; ++k) {
            acc[k] = false;
            key[k] = __builtin_inf();
        }
#pragma unroll
        for (int h = 0; h < kReg; h += BATCH) {
            if (!SKIP || h < n) {
                P64 q[BATCH];
#pragma unroll
                for (int e = 0; e < BATCH; ++e) q[e] = p.B[h + e < n ? j[h + e] : (SKIP ? j[h] : i)];
#pragma unroll
                for (int e = 0; e < BATCH; ++e) {
                    const int k = h + e;
                    const uint32_t c = w >> (6 * k);
                    const int wx = (int)(c & 3u) - 1, wy = (int)((c >> 2) & 3u) - 1, wz = (int)((c >> 4) & 3u) - 1;
                    double rx = q[e].x - me.x, ry = q[e].y - me.y, rz = q[e].z - me.z;
                    if (wx != 0) rx = rx + (double)wx * B.L[0];
                    if (wy != 0) ry = ry + (double)wy * B.L[1];
                    if (wz != 0) rz = rz + (double)wz * B.L[2];
                    const PairQ pq = pair_q(rx, ry, rz, q[e].vx - me.vx, q[e].vy - me.vy, q[e].vz - me.vz);
                    acc[k] = k < n && accept(pq, K ? pair_D2(p, B, row, j[k]) : B.D2, B.dt);
                    key[k] = acc[k] ? pq.c2 / pq.g2 : __builtin_inf();
                }
            }
        }
        double best_key = __builtin_inf();
        int32_t best = -1;
#pragma unroll
        for (int k = 0; k < kReg; ++k) {
            if (acc[k] && (best < 0 || key[k] < best_key ||
                           (key[k] == best_key && p.idB[j[k]] < p.idB[best]))) {
                best_key = key[k];
                best = (int32_t)j[k];
            }
        }
#pragma unroll
        for (int k = 0; k < kReg; ++k) {
            if (slot[k] < (uint32_t)kSlots) {
                SlotEntry e;
                e.key = acc[k] ? key[k] : __builtin_inf();
                e.j = i;
                e.pad_ = 0u;
                p.sl[(size_t)slot[k] * p.N + j[k]] = e;
            }
        }
        p.fb_key[i] = best_key;
        p.fb_j[i] = best;
        return (uint32_t)n;
    }
    // The wave's extra pairs: decided in FP64 and posted to both candidate
    // lists (tile0: the wave's first particle).
    __device__ __forceinline__ void flush_extra(const Plan& p, uint32_t tile0, uint32_t lane)
    {
        const uint32_t m = min(extra->n, kExtra);
        for (uint32_t t = lane; t < m; t += 64u) {
            const uint32_t a = tile0 + extra->lane[t], j = extra->j[t];
            const P64 me = p.B[a];
            double key;
            if (exact_key(p, box_of(p, a), a, me, j, key)) {
                post_candidate(p, a, j, key);
                post_candidate(p, j, a, key);
            }
        }
    }
};

// Per-group context of the FP64 search: the criteria's constants, in scalar
// registers (loaded per chunk they were waited for before its pair loop).
struct Group64 {
    double D2, dt;
};

__device__ __forceinline__ double uniform64(double x)
{
    const uint64_t b = (uint64_t)__double_as_longlong(x);
    const uint32_t lo = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)b);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(b >> 32));
    return __longlong_as_double((long long)((uint64_t)hi << 32 | lo));
}

// Running (key, id) minimum of one lane in the full-neighbourhood search.
struct Best {
    double key;
    float kcut;          // FP32 screen: folded constant of the m3 test for the best key so far
    uint32_t id;
    int32_t j;
    uint32_t accepted;   // acceptable pairs seen (statistics)
    uint32_t screened;   // FP32 screen: pairs it could not reject (statistics)
    __device__ __forceinline__ void clear()
    {
        key = __builtin_inf();
        // finite: its product with a g2 of zero (velocities equal in FP32 and not
        // in FP64) is zero, and the pair stays
        kcut = 0x1.fffffep127f;
        id = 0xFFFFFFFFu;
        j = -1;
        accepted = 0u;
        screened = 0u;
    }
    __device__ __forceinline__ void offer(double k, uint32_t idj, uint32_t jj)
    {
        if (k < key || (k == key && idj < id)) {
            key = k;
            id = idj;
            j = (int32_t)jj;
        }
    }
    // An acceptable pair: its key is divided out only if it can be the best
    // (a particle with many acceptable partners improves on its best a few
    // times, and every division stalls the whole wave).  c2 / g2 rounds to at
    // most key only if c2 <= key (1 + 2^-53) g2, or key is subnormal; the
    // comparison's own roundings are below its slack of 2^-50.
    __device__ __forceinline__ void take(const PairQ& q, uint32_t idj, uint32_t jj)
    {
        accepted += 1u;
        if (q.c2 * (1.0 - 0x1.0p-50) <= (key + 0x1.0p-1022) * q.g2) offer(q.c2 / q.g2, idj, jj);
    }
};

// Pairs of the full-neighbourhood search that the FP32 screen can neither
// reject nor show to be worse than the particle's best: decided in FP64 once
// the tile's rows are done (a record gather inside the pair loop stalls the
// whole wave).  Each waits with a lower bound on its key: when the slots are
// full, one that the best has overtaken makes room, and at the end only those
// that may still win are decided, whatever the number of partners.  A particle
// for which that is not enough (six pairs within the screen's error of each
// other) is searched again in FP64 by the whole wave.  Against four unpruned
// slots and an FP64 decision in the loop for every further pair: 1e7
// particles of one speed (11 partners each) 4.65 -> 2.38 ms, 1e7 in blobs (up
// to 180 partners) 15.9 -> 10.5 ms, 256 boxes (2.8 partners) 1.66 -> 1.53 ms,
// and no spilled registers; eight slots without the lower bounds, the
// overtaken pairs staying in them, took 18.9 ms on the blobs for the particles
// searched again.
constexpr int kDefer = 5;
// Up to this many particles of a tile the wave searches again itself, one after
// another (about 4 us each at three per cell).  More of them, where velocities
// are equal in FP32 and no pair can be told from another (beams, a gas at rest),
// go to the step's list (1e6 particles of one velocity: 1130 us a step by the
// waves themselves, 660 by the list, which gives way to the whole-step search).
// So do those of dense cells, with their thousands of candidates, in a gas of
// one round of waves, where each wave's time shows (1.8e5 in two clusters: 18.1
// -> 11.7 ms); in a larger gas other waves run beside it, and the list's few
// long searches would come after (1e7 in blobs: 180 to 410 us a step).
constexpr int kAgainAlone = 16;
constexpr uint32_t kAgainCell = 64;
constexpr uint32_t kAgainRound = 64u * 6u * 4u * 256u;   // six waves on each SIMD
struct DeferLds {
    uint32_t j[kDefer][64];      // sorted index
    float lo[kDefer][64];        // lower bound of the key
    uint8_t code[kDefer][64];    // image shift (wcode)
};
struct Deferred {
    DeferLds* l;
    int n;   // kDefer + 1: there were more
};

// Tile shape of a search kernel: W records staged per LDS chunk, and the
// waves per SIMD the half- and full-neighbourhood searches are compiled for
// (fewer waves leave more registers per wave).  The launch autotuner picks
// one of three shapes per precision (kmc_config.tile); the results do not
// depend on it.
template <int W_, int HALF_WAVES, int FULL_WAVES>
struct Tile {
    static constexpr int W = W_;
    static constexpr int kWaves = HALF_WAVES;
    static constexpr int kFullWaves = FULL_WAVES;
};
// FP64: 96 records per chunk (4.5 KiB) by default
using TileF64_0 = Tile<96, 6, 5>;
using TileF64_1 = Tile<64, 6, 5>;
using TileF64_2 = Tile<160, 5, 4>;
// FP32 screen: 128 records (4 KiB) by default (measured against 96, 160,
// 192 and 256 on the headline gas)
using TileF32_0 = Tile<128, 6, 5>;
using TileF32_1 = Tile<64, 6, 5>;
using TileF32_2 = Tile<256, 5, 4>;

// K: particles of several kinds (the pair's D2 from the per-kind-pair table,
// staged in LDS with each record's kind); otherwise the box's D2.
template <bool K, class T = TileF64_0>
struct PolF64 {
    static constexpr int W = T::W;
    static constexpr bool kScreen = false;
    static constexpr bool kKinds = K;
    static constexpr int kFlushBatch = 2;
    static constexpr bool kFlushSkipEmpty = true;
    static constexpr int kWaves = T::kWaves;
    static constexpr int kFullWaves = T::kFullWaves;
    struct Lds {
        P64 rec[W];
        uint8_t kind[K ? W : 1];
        double d2[K ? kMaxKinds * kMaxKinds : 1];
    };
    struct Own {
        P64 me;
        uint32_t row;   // K: kMaxKinds * own kind
    };
    using Group = Group64;
    __device__ static void begin_group(const Lds&, const Plan&, const BoxDev& B, Own&, Group& g, int, int, int, int, int,
                                       uint32_t, bool)
    {
        g.D2 = uniform64(B.D2);
        g.dt = uniform64(B.dt);
    }
    // per-group LDS tables, written before the group's first staging barrier
    __device__ static void group_lds(Lds& l, const Plan& p, uint32_t, int lane)
    {
        if (K) l.d2[lane] = p.sp_D2[lane];
    }
    __device__ static void load_own(Lds&, const Plan& p, uint32_t i, Own& o, double& x, double& y, double& z)
    {
        o.me = p.B[i];
        o.row = K ? (uint32_t)p.spB[i] * (uint32_t)kMaxKinds : 0u;
        x = o.me.x; y = o.me.y; z = o.me.z;
    }
    __device__ static P64 self64(const Plan&, uint32_t, const Own& o) { return o.me; }
    __device__ static void stage(Lds& l, uint32_t t, const Plan& p, uint32_t j, const BoxDev&, const Group&, int, int,
                                 int)
    {
        l.rec[t] = p.B[j];
        if (K) l.kind[t] = p.spB[j];
    }
    template <bool SH, class M>
    __device__ static void scan(const Lds& l, uint32_t c0, uint32_t j0, uint32_t j1, const Own& o, const BoxDev& B,
                                const Group& g, const M& m, Found& f)
    {
        const double sx = (double)m.wx * B.L[0], sy = (double)m.wy * B.L[1], sz = (double)m.wz * B.L[2];
        const double D2 = g.D2, dt = g.dt;
        for (uint32_t j = j0; j < j1; ++j) {
            const P64 q = l.rec[j - c0];
            double rx = q.x - o.me.x, ry = q.y - o.me.y, rz = q.z - o.me.z;
            if (SH) { rx = rx + sx; ry = ry + sy; rz = rz + sz; }
            const PairQ pq = pair_q(rx, ry, rz, q.vx - o.me.vx, q.vy - o.me.vy, q.vz - o.me.vz);
            const double d2 = K ? l.d2[o.row + l.kind[j - c0]] : D2;
            if (accept(pq, d2, dt)) f.add(j, m);
        }
    }
    // full neighbourhood: running (key, id) minimum over the acceptable pairs
    // (the particle itself has g2 = 0 and is never accepted)
    template <bool SH, class M>
    __device__ static void scan_best(const Lds& l, const uint32_t* lid, uint32_t c0, uint32_t j0, uint32_t j1, uint32_t,
                                     const Own& o, const BoxDev& B, const Group& g, const M& m, Best& best, Deferred&)
    {
        const double sx = (double)m.wx * B.L[0], sy = (double)m.wy * B.L[1], sz = (double)m.wz * B.L[2];
        const double D2 = g.D2, dt = g.dt;
        for (uint32_t j = j0; j < j1; ++j) {
            const P64 q = l.rec[j - c0];
            double rx = q.x - o.me.x, ry = q.y - o.me.y, rz = q.z - o.me.z;
            if (SH) { rx = rx + sx; ry = ry + sy; rz = rz + sz; }
            const PairQ pq = pair_q(rx, ry, rz, q.vx - o.me.vx, q.vy - o.me.vy, q.vz - o.me.vz);
            const double d2 = K ? l.d2[o.row + l.kind[j - c0]] : D2;
            if (accept(pq, d2, dt)) best.take(pq, lid[j - c0], j);
        }
    }
};

// FP32 screen.  Positions are rounded to FP32 relative to the centre X0 of
// the group's neighbourhood (periodic images added in FP64 first), so their
// rounding error is u times the neighbourhood size, not the box size.  The
// screen tests the Lagrange form d_min^2 g2 = |r|^2 g2 - b^2 (cheaper than the
// cross product) and drops a pair only when the FP64 definition is certain to
// reject it; every pair it keeps is decided exactly in FP64 afterwards.
//
// The bounds depend on how far a group's neighbourhood reaches along x.  A
// screened group of at most span_cells(c) cells uses the thresholds of class
// c (k_step_setup computes each class per box), so dense rows keep tight
// bounds while the lanes of a sparse row (under one particle per cell),
// hundreds of cells apart, share looser ones; the search splits rows wider
// than the last class.
__host__ __device__ constexpr int span_cells(int c) { return 64 << (2 * c); }
constexpr int kScreenGroupCells = span_cells(kSpanClasses - 1);

__device__ __forceinline__ uint32_t span_class(int cells)
{
    uint32_t c = 0;
    while (c + 1 < (uint32_t)kSpanClasses && cells > span_cells((int)c)) ++c;
    return c;
}

struct ScreenGroup {
    double X0[3];
    ScreenBounds t;
};

// Bounds on |screen value - FP64 definition value| for every neighbour pair
// of any search group of the box (forward error analysis, Higham 2002,
// ch. 3).  Inputs: |r_k| <= R_k = 2 h_k; FP32 position errors
// e_r,k = u (2 P_k + 2 R_k) with positions relative to the group centre X0
// (a group of class c spans at most s = span_cells(c) cells along x, so
// |x - X0| <= P_x = (s/2 + 1) h_x, P_y = 1.5 h_y, P_z = 1.5 h_z) plus the
// FP64 definition's own input rounding; velocity-difference error
// e_g = 4 u V.
// With q = sqrt(g2_hat) (kappa q bounds every |g_hat_k|):
//   |db|   <= b0 + b1 q
//   |dg2|  <= g0 + g1 q + g2c q^2
//   |dm2|  <= P0 + P1 q + P2 q^2          (m2 = -b - dt g2)
//   |dm3|  <= A0 + A1 q + A2 q^2          (m3 = (|r|^2 - D2) g2 - b^2, Lagrange form
//                                          of the definition's c2 - D2 g2)
// and q <= (q^2 / G0 + G0) / 2 for any G0 > 0 makes each bound affine in
// g2_hat.  gamma terms cover the rounding of every sum and product in both
// precisions; the guard factor scales the result.
// The bound itself, for a screen of unit roundoff u: er[k] bounds the error
// of the screen's r_k (including the FP64 definition's own input rounding),
// R[k] bounds |r_k|, eg the error of each g_k, D2 and dt are the criteria's
// constants in the screen's units, G0 > 0 the AM-GM point, f the guard
// factor.  t = {b0, b1, t0, t1, c0, c1, g0, g1} of the affine thresholds.
__device__ __forceinline__ void screen_bound(double u, const double er[3], const double Rk[3], double eg, double D2,
                                             double dt, double G0, double f, double t[8])
{
    const double u64 = 0x1.0p-53;
    const double g3 = 3.0 * u / (1.0 - 3.0 * u) + 3.0 * u64 / (1.0 - 3.0 * u64);
    const double kap = 1.0 + g3;
    double SE = 0, SRE = 0, RR = 0, Err = 0;
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        SE += er[k];
        SRE += Rk[k] + er[k];
        RR += (Rk[k] + er[k]) * (Rk[k] + er[k]);
        Err += 2.0 * Rk[k] * er[k] + er[k] * er[k];
    }
    Err += g3 * RR;
    const double Rn = sqrt(RR) * (1.0 + 1e-12);
    const double s3 = 1.7320508075688774;     // >= sqrt(3)
    const double b0 = eg * (SRE + SE), b1 = kap * (SE + g3 * SRE);
    const double g0 = 3.0 * eg * eg, g1 = 2.0 * s3 * kap * eg, g2c = g3 * kap * kap;
    const double Et = Err + u * D2 + 6.0 * u * (RR + D2);
    const double Tm = RR + D2 + Et;
    const double A2 = 2.0 * Rn * kap * b1 + b1 * b1 + u * RR * kap * kap * (1.0 + g3) * (1.0 + g3) + Tm * g2c +
                      Et * (1.0 + g2c) + 128.0 * u64 * (RR + D2) * kap * kap;
    const double A1 = 2.0 * Rn * (kap * b0 + s3 * eg * b1) + 2.0 * b0 * b1 + Tm * g1 + Et * g1;
    const double A0 = 2.0 * Rn * s3 * eg * b0 + b0 * b0 + Tm * g0 + Et * g0 + 384.0 * u64 * (RR + D2) * eg * eg;
    const double dtf = dt * (1.0 + 2.0 * u64);
    const double P0 = b0 + dtf * g0, P1 = b1 + dtf * g1, P2 = dtf * g2c + (u + u64) * dt;
    t[0] = f * (b0 + 0.5 * b1 * G0);
    t[1] = f * (0.5 * b1 / G0);
    t[2] = f * (P0 + 0.5 * P1 * G0);
    t[3] = f * (P2 + 0.5 * P1 / G0);
    t[4] = f * (A0 + 0.5 * A1 * G0);
    t[5] = f * (A2 + 0.5 * A1 / G0);
    t[6] = f * (g0 + 0.5 * g1 * G0);
    t[7] = f * (g2c + 0.5 * g1 / G0);
}

// Folded D2 constant of the m3 test for the criterion's FP32 D2 (see below).
__device__ __forceinline__ float fold_kD2(double D2_32, double tc1, double RRb)
{
    const double u = 0x1.0p-24;
    return tc1 > 0.0 ? (float)((D2_32 + tc1 + 6.0 * u * (RRb + D2_32 + tc1)) * (1.0 + 2e-6)) : (float)D2_32;
}

// Returns the g2 slopes tt1 and tc1 and RRb (for fold_kD2 with other D2 values of the box).  With
// particle kinds B.D2 is the largest pair value; every bound term grows with
// D2, so the bounds hold for every pair of kinds.
__device__ __forceinline__ void screen_thresholds(const BoxDev& B, const double P[3], double V, float guard,
                                                  ScreenBounds& g, double& tt1, double& tc1, double& RRb)
{
    const double u = 0x1.0p-24, u64 = 0x1.0p-53;
    const double eg = 4.0001 * u * V + 4.0 * u64 * V;
    double er[3], Rk[3];
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        Rk[k] = B.rmax[k];
        er[k] = u * (2.0 * P[k] + 2.0 * Rk[k]) * (1.0 + 1e-5) + 2.0 * u64 * (Rk[k] + 2.0 * B.L[k]);
    }
    const double G0 = V > 0.0 ? 0.25 * V : 1.0;
    const double f = (double)guard * (1.0 + 1e-5) * (1.0 + 1e-6);
    double t[8];
    screen_bound(u, er, Rk, eg, B.D2, B.dt, G0, f, t);
    // thresholds rounded to FP32 stay above the bounds (f carries 1e-5 of slack)
    g.tb0 = (float)t[0];
    g.tb1 = (float)t[1];
    g.tt0 = (float)t[2];
    // The relative bounds do not see products that underflow: b^2 and the last
    // product of the m3 test each lose up to 2^-150 (the errors that underflow
    // leaves in b and g2 are a small fraction of the bounds for edges and speeds
    // of at least 2^-40, where tc0 is 2^-180 or more).  2^-140 covers them, also
    // in the pruning's use of tc.
    g.tc0 = (float)t[4] + 0x1p-140f;
    // Folded constants, rounded up (the factor 1 + 2e-6 exceeds every rounding
    // here).  m2: -b - kdt g2 <= -b - (dt + tt1) g2 for kdt >= dt + tt1, and the
    // screen's one rounding of the FMA is monotone.  m3: the screen sums
    // |r|^2 - D2 in three FMAs that start from -D2, each with an error of at most
    // u (|r|^2 + D2); replacing D2 by kD2 lowers the sum by at least kD2 - D2 less
    // the errors of both, which is >= tc1 when kD2 (1 - 3 u) >= D2 (1 + 3 u) +
    // tc1 + 6 u RRb with RRb >= |r|^2.
    // Without bounds (guard 0) the constants are the criteria's own.
    const double dt32 = (double)B.dt_32;
    RRb = 0.0;
#pragma unroll
    for (int k = 0; k < 3; ++k) RRb += (Rk[k] + er[k]) * (Rk[k] + er[k]);
    RRb *= 1.0 + 1e-5;
    tt1 = t[3];
    tc1 = t[5];
    g.kdt = t[3] > 0.0 ? (float)((dt32 + t[3]) * (1.0 + 2e-6)) : B.dt_32;
    g.kD2 = fold_kD2((double)B.D2_32, t[5], RRb);
    // Pruning by the best key of a particle (full search).  A pair whose key
    // is at most K passes the m3 test with the constant folded for K, by the
    // same argument as for D2 (the bounds grow with D2, and K < D2): kc is the
    // part of that constant that does not depend on K; the factor 1 + 4e-6 on
    // K and on kc exceeds the rounding of K to FP32 and of the sum.  A pair is
    // certain to be acceptable when it passes the tests with the bounds on the
    // other side (kdm <= dt - tt1, g2 above its own error), and its key is
    // then at most |r|^2 + tc1 - (b^2 - tc0) / g2, which has to be below D2
    // (taken from kD2: D2 >= (1 - 5e-6) kD2 - kc).  The factor 1 + 1e-6 on |r|^2
    // exceeds the rounding of the quotient (b^2 / g2 is at most |r|^2), and a
    // second tc1 (tcu is twice tc1) that of |r|^2, which is summed as (|r|^2 -
    // kD2) + kD2 with errors of at most 6 u (RRb + kD2).  In the same way
    // |r|^2 (1 - 1e-6) - tcu - (b^2 + tc0) / g2 is no larger than the K at which the
    // pair would fail the folded test.
    g.kc = (float)((t[5] + 6.0 * u * (RRb + t[5])) * (1.0 + 4e-6));
    g.tcu = (float)(2.0 * t[5] * (1.0 + 2e-6));
    // The tests on b and m2 as one: -(g + kdt g2) <= b <= g + tb1 g2 with g the
    // larger of tb0 and tt0 is |b + ka g2| <= g + kb g2 (ka, kb half the
    // difference and half the sum); the factor 1 + 1e-6 on kb and g exceeds
    // the rounding of both sides and makes the inequality strict, so that the
    // sign bit of their difference decides.
    g.ka = 0.5f * (g.kdt - g.tb1);
    g.kb = 0.5f * (g.kdt + g.tb1) * 1.000001f;
    g.kg = fmaxf(g.tb0, g.tt0) * 1.000001f;
    g.tc = g.tc0 * 1.000001f;
    // Nothing is acceptable in a gas at rest, and no pair passes (with b = g2 = 0
    // every one would, and end in the re-search).
    if (V == 0.0) g.tb0 = g.kg = -1.0f;
    g.kdm = (float)((dt32 - t[3]) * (1.0 - 2e-6));
    g.gmin = t[7] < 0.5 ? (float)(2.0 * t[6] * (1.0 + 2e-6)) : __builtin_inff();
}

// The thresholds of span class c of box b for the largest speed V, computed by
// a whole wave (with particle kinds each lane folds the constant of one pair
// of kinds); true in every lane when the screen is safe to use.
//
// The bounds take FP32 arithmetic to neither overflow nor lose to underflow
// more than a small fraction of them (beside what tc0 allows for): cell edges in [2^-40, 2^40], the largest
// speed 0 or in [2^-40, 2^40], the pair test's largest products (|r|^2 g2 <=
// 144 h^2 V^2 and the folded thresholds times g2 <= 12 V^2) below 2^120, every
// threshold finite.  Outside that range this step's partners come from the
// whole-step FP64 search.
__device__ __forceinline__ bool screen_class(const Plan& p, const BoxDev& B, uint32_t b, int c, double V, int lane,
                                             bool store)
{
    const double lo_s = 0x1.0p-40, hi_s = 0x1.0p40, big = 0x1.0p120;
    bool safe = V == 0.0 || (V >= lo_s && V <= hi_s);
    double hmax = 0.0;
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        safe = safe && B.h[k] >= lo_s && B.h[k] <= hi_s;
        hmax = fmax(hmax, B.h[k]);
    }
    const double g2max = 12.0 * V * V;
    safe = safe && 256.0 * hmax * hmax * g2max < big;
    // neighbourhood of a group of this class in cells (its own cells and one
    // on each side)
    const double cells[3] = {(double)(span_cells(c) + 2), 3.0, 3.0};
    double P[3];
#pragma unroll
    for (int k = 0; k < 3; ++k)
        P[k] = 0.5 * cells[k] * B.h[k] * (1.0 + 1e-9) + 1e-12 * (fabs(B.lo[k]) + fabs(B.hi[k]) + 2.0 * B.L[k]);
    double tt1, tc1, RRb;
    ScreenBounds g;
    screen_thresholds(B, P, V, p.guard, g, tt1, tc1, RRb);
    if (store && lane == 0) p.box_sb[(size_t)b * kSpanClasses + c] = g;
    const float th[11] = {g.tb0, g.tb1, g.tt0, (float)tt1, g.tc0, (float)tc1, g.kdt, g.kD2, g.kc, g.kb, g.kg};
#pragma unroll
    for (int k = 0; k < 11; ++k) safe = safe && isfinite(th[k]) && (double)fabsf(th[k]) * g2max < big;
    if (p.nspecies > 0) {
        // the folded constant of each pair of kinds, from the pair's own D2
        // rounded to FP32 (entries of absent kinds are never read)
        static_assert(kMaxKinds * kMaxKinds == 64, "one lane per pair of kinds");
        const float kd = fold_kD2((double)(float)p.sp_D2[lane], tc1, RRb);
        if (store) p.box_kD2[((size_t)b * kSpanClasses + c) * (kMaxKinds * kMaxKinds) + (uint32_t)lane] = kd;
        safe = safe && isfinite(kd) && (double)kd * g2max < big;
    }
    return __ballot(safe) == ~0ull;
}

// What a step needs to know of every box before its search (one block per
// box, one wave per span class): the time step under the adaptive rule, dt =
// min(cap, (C dx) / sqrt(max |v|^2)), and the FP32 screen's thresholds.
// ALONE: the scatter blocks' partials are folded here (else by
// k_fold_partials).
template <bool ALONE>
__global__ __launch_bounds__(64 * kSpanClasses) void k_step_setup(Plan p)
{
    static_assert(kSpanClasses == 4, "fold_partials works in four waves");
    __shared__ float vmax;
    const uint32_t b = blockIdx.x;
    BoxDev& B = p.boxes[b];
    unsigned long long v2 = 0ull;
    float vm = 0.f;
    if (ALONE) fold_partials(p, B, threadIdx.x, blockDim.x, v2, vm);
    if (threadIdx.x == 0) {
        if (p.dt_rule == KMC_DT_ADAPTIVE) {
            const unsigned long long o = p.box_v2[b];
            p.box_v2[b] = 0ull;
            const double dt = adaptive_dt(p, B, o > v2 ? o : v2);
            B.dt = dt;
            B.dt_32 = (float)dt;
        }
        vmax = ALONE ? vm : __uint_as_float(p.box_vmax[b]);
    }
    __syncthreads();   // (the box's dt, too)
    if (p.precision != KMC_FP32_SCREEN) return;
    const double V = (double)vmax * (1.0 + 3.0 * 0x1.0p-24);
    const int lane = threadIdx.x & 63;
    const bool safe = screen_class(p, B, b, (int)(threadIdx.x >> 6), V, lane, true);
    if (!safe && lane == 0) atomicOr(&p.ctl->overflow, 1u);
}

// a < 0 and b < 0 (neither is NaN), by their sign bits: one comparison.  FP32
// sums, products and logic on vector registers issue at twice the rate of
// comparisons and of anything with a scalar operand here (measured 1.5 to 1.75
// against 0.9 instructions per CU and cycle), so a test that costs one
// comparison instead of three is worth the subtraction and the AND (with the
// 24-byte records and the shorter path of a kept pair: full search of 256
// boxes 1.53 -> 1.42 ms, of 1e7 particles of one speed 2.39 -> 2.30).
__device__ __forceinline__ bool both_negative(float a, float b)
{
    return (int)(__float_as_uint(a) & __float_as_uint(b)) < 0;
}

// K: particles of several kinds (the screen's folded D2 constant of each
// pair of kinds from a per-box table in LDS); otherwise the box's constant.
template <bool K, class T = TileF32_0>
struct PolF32 {
    static constexpr int W = K ? T::W * 3 / 4 : T::W;   // (with kinds, 24 waves would not fit a CU's LDS)
    static constexpr bool kScreen = true;
    static constexpr bool kKinds = K;
    static constexpr int kFlushBatch = 2;
    static constexpr bool kFlushSkipEmpty = true;
    static constexpr int kWaves = T::kWaves;
    static constexpr int kFullWaves = T::kFullWaves;
    // A staged candidate lies in two arrays: a = x, y, z relative to the group
    // centre and vx; b = vy, vz; its kind (particles of several kinds) in a
    // third.  Consecutive records fall in distinct LDS banks, and two of them
    // are read by three instructions.
    struct Lds {
        float4 a[W];
        float2 b[W];
        uint8_t kind[K ? W : 1];
        double own[3][K ? 64 : 1];
        float kd2[K ? kMaxKinds * kMaxKinds : 1];
    };
    struct Own {
        float x, y, z, vx, vy, vz;   // position relative to the current group's centre
        uint32_t row;                // K: kMaxKinds * own kind
        double X, Y, Z;              // own FP64 position (kept: reloading it per group costs more;
                                     // with kinds in LDS, where it would spill)
    };
    using Group = ScreenGroup;
    __device__ static P64 self64(const Plan& p, uint32_t i, const Own&) { return p.B[i]; }
    __device__ static void load_own(Lds& l, const Plan& p, uint32_t i, Own& o, double& x, double& y, double& z)
    {
        const P64 m = p.B[i];
        o.vx = (float)m.vx; o.vy = (float)m.vy; o.vz = (float)m.vz;
        o.row = K ? (uint32_t)p.spB[i] * (uint32_t)kMaxKinds : 0u;
        x = m.x; y = m.y; z = m.z;
        if (K) {
            l.own[0][threadIdx.x] = m.x;
            l.own[1][threadIdx.x] = m.y;
            l.own[2][threadIdx.x] = m.z;
        } else {
            o.X = m.x; o.Y = m.y; o.Z = m.z;
        }
    }
    // per-group LDS tables, written before the group's first staging barrier
    // (sbi: the group's threshold set, box * kSpanClasses + span class)
    __device__ static void group_lds(Lds& l, const Plan& p, uint32_t sbi, int lane)
    {
        if (K) l.kd2[lane] = p.box_kD2[(size_t)sbi * (kMaxKinds * kMaxKinds) + (uint32_t)lane];
    }
    // Centre and thresholds (set sbi) of the group whose cells are x in
    // [cxf, cxl] of row (gcy, gcz); its neighbourhood spans cells
    // cxf-1..cxl+1, gcy-1..gcy+1, gcz-1..gcz+1 (images included).
    __device__ static void group_ctx(const Plan& p, const BoxDev& B, Group& g, int cxf, int cxl, int gcy, int gcz,
                                     int sbi)
    {
        const int clo[3] = {cxf - 1, gcy - 1, gcz - 1}, chi[3] = {cxl + 1, gcy + 1, gcz + 1};
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            const double h = B.h[k];
            g.X0[k] = B.lo[k] + 0.5 * (double)(clo[k] + chi[k] + 1) * h;
        }
        g.t = p.box_sb[sbi];
    }
    __device__ static void begin_group(const Lds& l, const Plan& p, const BoxDev& B, Own& o, Group& g, int cxf, int cxl,
                                       int gcy, int gcz, int sbi, uint32_t i, bool in)
    {
        group_ctx(p, B, g, cxf, cxl, gcy, gcz, sbi);
        if (in) {
            const uint32_t t = K ? threadIdx.x : 0u;
            o.x = (float)((K ? l.own[0][t] : o.X) - g.X0[0]);
            o.y = (float)((K ? l.own[1][t] : o.Y) - g.X0[1]);
            o.z = (float)((K ? l.own[2][t] : o.Z) - g.X0[2]);
        }
    }
    // FP32 copy of a candidate: image-shifted position relative to X0 and
    // velocity, each rounded once.  Rows without an image (almost all) skip
    // the shift (the row's shift is the same for the whole wave).
    __device__ static void stage(Lds& l, uint32_t t, const Plan& p, uint32_t j, const BoxDev& B, const Group& g,
                                 int wx, int wy, int wz)
    {
        const P64 q = p.B[j];
        double x = q.x, y = q.y, z = q.z;
        if (wx | wy | wz) {
            x = x + (wx ? (double)wx * B.L[0] : 0.0);
            y = y + (wy ? (double)wy * B.L[1] : 0.0);
            z = z + (wz ? (double)wz * B.L[2] : 0.0);
        }
        l.a[t] = make_float4((float)(x - g.X0[0]), (float)(y - g.X0[1]), (float)(z - g.X0[2]), (float)q.vx);
        l.b[t] = make_float2((float)q.vy, (float)q.vz);
        if (K) l.kind[t] = p.spB[j];
    }
    template <bool SH, class M>
    __device__ static void scan(const Lds& l, uint32_t c0, uint32_t j0, uint32_t j1, const Own& o, const BoxDev&,
                                const Group& g, const M& m, Found& f)
    {
        const float ka = g.t.ka, kb = g.t.kb, kg = g.t.kg, tc = g.t.tc, kD2 = g.t.kD2;
        // the loop steps LDS pointers only; a kept pair's sorted index comes
        // from the pointer
        const float4* pa = l.a + (j0 - c0);
        const float2* pb = l.b + (j0 - c0);
        const float4* const pe = pa + (j1 > j0 ? j1 - j0 : 0u);
        auto test = [&](const float4& qa, const float2& qb, uint32_t t) {
            const float rx = qa.x - o.x, ry = qa.y - o.y, rz = qa.z - o.z;
            const float gx = qa.w - o.vx, gy = qb.x - o.vy, gz = qb.y - o.vz;
            const float kd = K ? l.kd2[o.row + l.kind[t]] : kD2;
            const float b = fmaf(rz, gz, fmaf(ry, gy, rx * gx));
            const float g2 = fmaf(gz, gz, fmaf(gy, gy, gx * gx));
            const float rk = fmaf(rz, rz, fmaf(ry, ry, fmaf(rx, rx, -kd)));   // |r|^2 - kd
            return both_negative(fabsf(fmaf(ka, g2, b)) - fmaf(kb, g2, kg), fmaf(rk, g2, fmaf(-b, b, -tc)));
        };
        // two records per iteration: one loop test and one branch on the
        // kept pairs per two pair tests, and all LDS reads in flight
        for (; pa + 1 < pe; pa += 2, pb += 2) {
            const float4 qa0 = pa[0], qa1 = pa[1];
            const float2 qb0 = pb[0], qb1 = pb[1];
            const uint32_t t = K ? (uint32_t)(pa - l.a) : 0u;
            const bool k0 = test(qa0, qb0, t), k1 = test(qa1, qb1, t + 1u);
            if (k0 | k1) f.add2(k0, k1, c0 + (uint32_t)(pa - l.a), m);
        }
        if (pa < pe) {
            const float4 qa = pa[0];
            const float2 qb = pb[0];
            if (test(qa, qb, K ? (uint32_t)(pa - l.a) : 0u)) f.add(c0 + (uint32_t)(pa - l.a), m);
        }
    }
    // full neighbourhood: every pair the screen cannot reject is decided in
    // FP64 from the sorted records, with the image shift of its cell
    template <bool SH, class M>
    __device__ static void scan_best(const Lds& l, const uint32_t*, uint32_t c0, uint32_t j0, uint32_t j1, uint32_t i,
                                     const Own& o, const BoxDev&, const Group& g, const M& m, Best& best, Deferred& d)
    {
        const float ka = g.t.ka, kb = g.t.kb, kg = g.t.kg, tc = g.t.tc, kD2 = g.t.kD2;
        struct Q {
            float b, g2, rk;   // rk: |r|^2 - kd
        };
        auto test = [&](const float4& qa, const float2& qb, uint32_t t, Q& q) {
            const float rx = qa.x - o.x, ry = qa.y - o.y, rz = qa.z - o.z;
            const float gx = qa.w - o.vx, gy = qb.x - o.vy, gz = qb.y - o.vz;
            const float kd = K ? l.kd2[o.row + l.kind[t]] : kD2;
            q.b = fmaf(rz, gz, fmaf(ry, gy, rx * gx));
            q.g2 = fmaf(gz, gz, fmaf(gy, gy, gx * gx));
            q.rk = fmaf(rz, rz, fmaf(ry, ry, fmaf(rx, rx, -kd)));
            return both_negative(fabsf(fmaf(ka, q.g2, q.b)) - fmaf(kb, q.g2, kg),
                                 fmaf(q.rk, q.g2, fmaf(-q.b, q.b, -tc)));
        };
        // a kept pair: dropped if its key is certain to exceed the best so
        // far, else recorded for the end of the tile
        auto take = [&](uint32_t f, const Q& q) {
            uint32_t code;
            const uint32_t j = m.at(f, code);
            if (j == i) return;   // (the particle itself passes the tests)
            best.screened += 1u;
            const float kd = K ? l.kd2[o.row + l.kind[f - c0]] : kD2;
            const float bb = q.b * q.b;
            if (!(fmaf(q.rk + (kd - best.kcut), q.g2, -bb) <= tc)) return;
            // certain to be acceptable: its key's upper bound prunes from here on
            const float ig = __builtin_amdgcn_rcpf(q.g2), rr = q.rk + kd;
            const float ku = fmaf(rr, 1.000001f, g.t.tcu) + (tc - bb) * ig;
            if ((fmaf(g.t.tb1, q.g2, q.b) <= -g.t.tb0) & (fmaf(-g.t.kdm, q.g2, -q.b) <= -g.t.tt0) &
                (ku < fmaf(kd, 0.999995f, -g.t.kc)) & (q.g2 > g.t.gmin))
                best.kcut = fminf(best.kcut, fmaf(fmaxf(ku, 0.f), 1.000004f, g.t.kc));
            int k = d.n;
            if (k < kDefer) {
                ++d.n;
            } else {
                k = -1;
                for (int e = 0; e < kDefer; ++e)
                    if (d.l->lo[e][threadIdx.x] > best.kcut) k = e;
                if (k < 0) {
                    d.n = kDefer + 1;
                    return;
                }
            }
            d.l->j[k][threadIdx.x] = j;
            d.l->lo[k][threadIdx.x] = fmaf(rr, 0.999999f, -g.t.tcu) - (bb + tc) * ig;
            d.l->code[k][threadIdx.x] = (uint8_t)code;
        };
        const float4* pa = l.a + (j0 - c0);
        const float2* pb = l.b + (j0 - c0);
        const float4* const pe = pa + (j1 > j0 ? j1 - j0 : 0u);
        Q q0, q1;
        for (; pa + 1 < pe; pa += 2, pb += 2) {   // two records per iteration, as in scan
            const float4 qa0 = pa[0], qa1 = pa[1];
            const float2 qb0 = pb[0], qb1 = pb[1];
            const uint32_t t = K ? (uint32_t)(pa - l.a) : 0u;
            const bool k0 = test(qa0, qb0, t, q0), k1 = test(qa1, qb1, t + 1u, q1);
            if (k0 | k1) {
                const uint32_t j = c0 + (uint32_t)(pa - l.a);
                if (k0) take(j, q0);
                if (k1) take(j + 1u, q1);
            }
        }
        if (pa < pe) {
            const float4 qa = pa[0];
            const float2 qb = pb[0];
            if (test(qa, qb, K ? (uint32_t)(pa - l.a) : 0u, q0)) take(c0 + (uint32_t)(pa - l.a), q0);
        }
    }
    // the deferred pairs of particle i, decided in FP64 with their image shifts
    __device__ static void decide_deferred(const Plan& p, uint32_t i, const Deferred& d, const BoxDev& B,
                                           Best& best)
    {
        if (d.n == 0 || d.n > kDefer) return;
        const P64 me = p.B[i];
        const uint32_t row = kind_row(p, i);
        for (int k = 0; k < d.n; ++k) {
            if (d.l->lo[k][threadIdx.x] > best.kcut) continue;   // overtaken
            const uint32_t j = d.l->j[k][threadIdx.x];
            const uint32_t c = d.l->code[k][threadIdx.x];
            const int wx = (int)(c & 3u) - 1, wy = (int)((c >> 2) & 3u) - 1, wz = (int)((c >> 4) & 3u) - 1;
            const P64 q = p.B[j];
            double rx = q.x - me.x, ry = q.y - me.y, rz = q.z - me.z;
            if (wx != 0) rx = rx + (double)wx * B.L[0];
            if (wy != 0) ry = ry + (double)wy * B.L[1];
            if (wz != 0) rz = rz + (double)wz * B.L[2];
            const PairQ pq = pair_q(rx, ry, rz, q.vx - me.vx, q.vy - me.vy, q.vz - me.vz);
            if (accept(pq, pair_D2(p, B, row, j), B.dt)) best.take(pq, p.idB[j], j);
        }
    }
};

// A row of a search group's neighbourhood: its window of cells (the same for
// the whole wave), the lane's part of it, and the row's image.
struct RowRange {
    uint32_t gs, ge;
    uint32_t ls, le;
    uint32_t row;
    int wy, wz;
    bool ok;
};

// A row's candidates, part by part: part(row, first f, end f, and the lane's
// own [lf, le)).  On a periodic x axis the cells beyond the ends of the row are
// the wrapped end cells, for the lanes at that end (back: the one before the
// first cell as well).  Taken as parts of their own they cost a staging and two
// barriers for one or two lanes' tests, and in a box of few cells along x most
// groups have them.  So the screen, whose records are staged with their image,
// takes them in one sequence with the row (256 uneven boxes in a context, 3 to
// a bin: full search 1.42 -> 1.32 ms; 1e5 in a box of 32^3 bins: half search
// 44.8 -> 40.6 us).  Other groups keep the plain sequence, in code of its own
// (one code for both costs 3 to 5 % where nothing wraps), and so does FP64:
// there the image enters each pair's arithmetic, once for the whole part.
template <class Pol, class F>
__device__ __forceinline__ void row_parts(const Plan& p, const BoxDev& B, const RowRange& R, bool back, bool in, int cx,
                                          int cxf, int cxl, F&& part)
{
    const int NX = B.nc[0];
    const uint32_t gs = (uint32_t)__builtin_amdgcn_readfirstlane((int)R.gs);
    const uint32_t ge = (uint32_t)__builtin_amdgcn_readfirstlane((int)R.ge);
    const bool left = B.periodic[0] && back && cxf == 0, right = B.periodic[0] && cxl == NX - 1;
    const Row m{0, R.wy, R.wz};
    if constexpr (Pol::kScreen) {
        if (left || right) {
            const uint32_t first = p.start[R.row], second = p.start[R.row + 1u];
            const uint32_t last = p.start[R.row + (uint32_t)NX - 1u], end = p.start[R.row + (uint32_t)NX];
            WrappedRow w;
            w.gs = gs;
            w.nM = ge - gs;
            w.sL = (uint32_t)__builtin_amdgcn_readfirstlane((int)last);
            w.nL = left ? (uint32_t)__builtin_amdgcn_readfirstlane((int)(end - last)) : 0u;
            w.sR = (uint32_t)__builtin_amdgcn_readfirstlane((int)first);
            const uint32_t nR = right ? (uint32_t)__builtin_amdgcn_readfirstlane((int)(second - first)) : 0u;
            w.wy = R.wy;
            w.wz = R.wz;
            const uint32_t total = w.nL + w.nM + nR;
            uint32_t lf = 0u, le = 0u;
            if (in) {
                lf = left && cx == 0 ? 0u : R.ls - gs + w.nL;
                le = right && cx == NX - 1 ? total : R.le - gs + w.nL;
            }
            part(w, 0u, total, lf, le);
            return;
        }
        part(m, gs, ge, R.ls, R.le);
    } else {
        part(m, gs, ge, R.ls, R.le);
        // k = 0: the wrapped cell to the left, k = 1: to the right
        for (int k = 0; k < 2; ++k) {
            if (!(k == 0 ? left : right)) continue;
            const int wc = k == 0 ? NX - 1 : 0;
            const uint32_t s = (uint32_t)__builtin_amdgcn_readfirstlane((int)p.start[R.row + (uint32_t)wc]);
            const uint32_t e = (uint32_t)__builtin_amdgcn_readfirstlane((int)p.start[R.row + (uint32_t)wc + 1u]);
            const bool mine = in && cx == (k == 0 ? 0 : NX - 1);
            part(Row{k == 0 ? -1 : 1, R.wy, R.wz}, s, e, mine ? s : 0u, mine ? e : 0u);
        }
    }
}

template <class Pol>
__global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(Pol::kWaves)))
void k_search_half(Plan p)
{
    __shared__ typename Pol::Lds lds;
    const int lane = threadIdx.x;
    const uint32_t i = xcd_tile(blockIdx.x, gridDim.x) * 64u + (uint32_t)lane;
    const bool valid = i < p.N;
    const bool alive = valid && !(p.idB[i] & kGone);   // absorbed particles do not search
    uint32_t bidx = 0, rowkey = 0xFFFFFFFFu;
    int cx = 0, cy = 0, cz = 0;
    typename Pol::Own own{};
    if (alive) {
        double x, y, z;
        Pol::load_own(lds, p, i, own, x, y, z);
        // (one box: its parameters are the same for every lane and come
        // through scalar loads, which keeps them out of the vector registers)
        auto locate = [&](const BoxDev& B) {
            cx = cell1(x, B.lo[0], B.inv_h[0], B.nc[0]);
            cy = cell1(y, B.lo[1], B.inv_h[1], B.nc[1]);
            cz = cell1(z, B.lo[2], B.inv_h[2], B.nc[2]);
            rowkey = B.coff + (uint32_t)B.nc[0] * ((uint32_t)cy + (uint32_t)B.nc[1] * (uint32_t)cz);
        };
        if (p.boxidx) {
            bidx = p.boxidx[i];
            locate(p.boxes[bidx]);
        } else {
            locate(p.boxes[0]);
        }
    }
    __shared__ uint32_t found_j[kReg * 64];
    __shared__ Extra extra;
    if (lane == 0) extra.n = 0u;   // (a barrier follows before the first pair is tested)
    Found found;
    found.clear(&extra, found_j + lane, p.sl_cnt);
    uint64_t remaining = __ballot(alive);
    while (remaining) {
        const int lead = __ffsll((unsigned long long)remaining) - 1;
        const uint32_t key = (uint32_t)__builtin_amdgcn_readlane((int)rowkey, lead);
        const int cxf = __builtin_amdgcn_readlane(cx, lead);
        // the row's lanes in ascending cells; a screened group ends after
        // kScreenGroupCells cells (the rest of the row forms the next one),
        // and its span picks its class of screen thresholds
        const uint64_t grp =
            __ballot(alive && rowkey == key && (!Pol::kScreen || cx - cxf < kScreenGroupCells)) & remaining;
        remaining &= ~grp;
        const bool in = (grp >> lane) & 1ull;
        const int last = 63 - __clzll((long long)grp);
        const uint32_t gb = (uint32_t)__builtin_amdgcn_readlane((int)bidx, lead);
        const BoxDev& B = p.boxes[gb];
        const int gcy = __builtin_amdgcn_readlane(cy, lead), gcz = __builtin_amdgcn_readlane(cz, lead);
        const int cxl = __builtin_amdgcn_readlane(cx, last);
        const int NX = B.nc[0], NY = B.nc[1], NZ = B.nc[2];
        typename Pol::Group gctx;
        const uint32_t sbi = gb * (uint32_t)kSpanClasses + span_class(cxl - cxf + 1);
        Pol::begin_group(lds, p, B, own, gctx, cxf, cxl, gcy, gcz, (int)sbi, i, in);
        Pol::group_lds(lds, p, sbi, lane);
        // The candidates [fs, fe) of a row; each lane tests those in [lf, le).
        auto part = [&](const auto& m, uint32_t fs, uint32_t fe, uint32_t lf, uint32_t le) {
            for (uint32_t c0 = fs; c0 < fe; c0 += (uint32_t)Pol::W) {
                const uint32_t n = min((uint32_t)Pol::W, fe - c0);
                for (uint32_t t = (uint32_t)lane; t < n; t += 64u) {
                    int wx;
                    const uint32_t j = m.at(c0 + t, wx);
                    Pol::stage(lds, t, p, j, B, gctx, wx, m.wy, m.wz);
                }
                __syncthreads();
                const uint32_t f0 = max(lf, c0), f1 = min(le, c0 + n);
                // (the screen's records are staged with their image shift)
                bool shift = false;
                if constexpr (!Pol::kScreen) shift = (m.wx | m.wy | m.wz) != 0;
                if (shift) Pol::template scan<true>(lds, c0, f0, f1, own, B, gctx, m, found);
                else Pol::template scan<false>(lds, c0, f0, f1, own, B, gctx, m, found);
                __syncthreads();
            }
        };
        // Rows of the half neighbourhood: the own one (from the particle on,
        // through cell cx+1), then (dy, dz) = (+1, 0), (-1, +1), (0, +1),
        // (+1, +1) with the cells cx-1..cx+1.  The ranges of a row are loaded
        // while the one before it is worked on (1e8 particles: 8.06 -> 7.82 ms,
        // the shock tube 82 -> 79 us; the full search has no registers to spare
        // for it: 1.42 -> 1.49 ms on 256 boxes).
        auto fetch = [&](int r, RowRange& R) {
            const int dy = r < 2 ? r : r - 3, dz = r < 2 ? 0 : 1;
            int nz = gcz + dz, ny = gcy + dy;
            R.wy = R.wz = 0;
            R.ok = r < 5;
            if (nz >= NZ) { R.ok = R.ok && B.periodic[2]; nz -= NZ; R.wz = 1; }
            if (ny < 0) { R.ok = R.ok && B.periodic[1]; ny += NY; R.wy = -1; }
            else if (ny >= NY) { R.ok = R.ok && B.periodic[1]; ny -= NY; R.wy = 1; }
            R.row = B.coff + (uint32_t)NX * ((uint32_t)ny + (uint32_t)NY * (uint32_t)nz);
            R.ls = R.le = 0;
            if (!R.ok) return;
            R.gs = p.start[R.row + (uint32_t)(r == 0 ? cxf : (cxf > 0 ? cxf - 1 : 0))];
            R.ge = p.start[R.row + (uint32_t)(cxl + 1 < NX ? cxl + 1 : NX - 1) + 1u];
            if (in) {
                R.ls = r == 0 ? i + 1u : p.start[R.row + (uint32_t)(cx > 0 ? cx - 1 : 0)];
                R.le = p.start[R.row + (uint32_t)(cx + 1 < NX ? cx + 1 : NX - 1) + 1u];
            }
        };
        RowRange R;
        fetch(0, R);
#pragma unroll 1
        for (int r = 0; r < 5; ++r) {
            RowRange next;
            fetch(r + 1, next);
            if (R.ok) row_parts<Pol>(p, B, R, r != 0, in, cx, cxf, cxl, part);
            R = next;
        }
    }
    uint32_t c = valid ? found.template flush<Pol::kFlushBatch, Pol::kFlushSkipEmpty, Pol::kKinds>(p, i, Pol::self64(p, i, own),
                                                                                       p.boxes[bidx])
                       : 0u;
    if (found.w >> 31) (void)atomicAdd(&p.sl_cnt[i], kMarked);
    __syncthreads();   // every lane's extra pairs are in LDS
    if (lane == 0) c += extra.n;
    found.flush_extra(p, xcd_tile(blockIdx.x, gridDim.x) * 64u, (uint32_t)lane);
    // statistics: pairs the search kept, counted at both particles
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) c += __shfl_xor(c, off, 64);
    if (lane == 0 && c) atomicAdd(&p.acc[blockIdx.x % p.acc_lanes].cand, 2ull * (unsigned long long)c);
}

// The FP64 search of one particle by a whole wave: lanes 0..26 look up one
// neighbouring cell each, the lanes share the candidates of all of them and
// the wave takes the (key, id) minimum.  (Row by row, each row's cell starts
// and records wait for the row before: 18 us for the few particles of a
// 1e5-particle step, now 7.5.)  All lanes of the wave must call it with
// the same i; returns the partner in every lane.
__device__ int32_t search_one64_wave(const Plan& p, uint32_t i)
{
    if (p.idB[i] & kGone) return -1;
    const int lane = threadIdx.x & 63;
    const BoxDev& B = box_of(p, i);
    const P64* __restrict__ X = p.B;
    const P64 me = X[i];
    const double dt = B.dt;
    const uint32_t row = kind_row(p, i);
    // this lane's neighbouring cell: its range of sorted particles and image
    uint32_t s = 0, n = 0, code = kNoImage;
    if (lane < 27) {
        const double xs[3] = {me.x, me.y, me.z};
        const int d[3] = {lane % 3 - 1, (lane / 3) % 3 - 1, lane / 9 - 1};
        int q[3], w[3];
        bool ok = true;
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            q[a] = cell1(xs[a], B.lo[a], B.inv_h[a], B.nc[a]) + d[a];
            w[a] = 0;
            if (q[a] < 0) { ok = ok && B.periodic[a]; q[a] += B.nc[a]; w[a] = -1; }
            else if (q[a] >= B.nc[a]) { ok = ok && B.periodic[a]; q[a] -= B.nc[a]; w[a] = 1; }
        }
        if (ok) {
            const uint32_t c = B.coff + (uint32_t)q[0] + (uint32_t)B.nc[0] * ((uint32_t)q[1] + (uint32_t)B.nc[1] * (uint32_t)q[2]);
            s = p.start[c];
            n = p.start[c + 1] - s;
            code = wcode(w[0], w[1], w[2]);
        }
    }
    uint32_t off = n;   // becomes the exclusive prefix of the range sizes
#pragma unroll
    for (int sft = 1; sft < 64; sft <<= 1) {
        const uint32_t y = __shfl_up(off, sft, 64);
        if (lane >= sft) off += y;
    }
    const uint32_t total = (uint32_t)__shfl((int)off, 63, 64);
    off -= n;
    double best_key = __builtin_inf();
    uint32_t best_id = 0xFFFFFFFFu;
    int32_t best = -1;
    for (uint32_t f0 = 0; f0 < total; f0 += 64u) {
        const uint32_t f = f0 + (uint32_t)lane;
        uint32_t r = 0;   // the last range that starts at or before candidate f
#pragma unroll
        for (uint32_t step = 16; step > 0; step >>= 1) {
            const uint32_t v = (uint32_t)__shfl((int)off, (int)(r + step), 64);
            if (r + step < 27u && v <= f) r += step;
        }
        const uint32_t j = (uint32_t)__shfl((int)s, (int)r, 64) + f - (uint32_t)__shfl((int)off, (int)r, 64);
        const uint32_t c = (uint32_t)__shfl((int)code, (int)r, 64);
        if (f < total) {
            const P64 q = X[j];
            const int wx = (int)(c & 3u) - 1, wy = (int)((c >> 2) & 3u) - 1, wz = (int)((c >> 4) & 3u) - 1;
            double rx = q.x - me.x, ry = q.y - me.y, rz = q.z - me.z;
            if (wx != 0) rx = rx + (double)wx * B.L[0];
            if (wy != 0) ry = ry + (double)wy * B.L[1];
            if (wz != 0) rz = rz + (double)wz * B.L[2];
            const PairQ pq = pair_q(rx, ry, rz, q.vx - me.vx, q.vy - me.vy, q.vz - me.vz);
            if (accept(pq, pair_D2(p, B, row, j), dt)) {
                const double key = pq.c2 / pq.g2;
                const uint32_t idj = p.idB[j];
                if (key < best_key || (key == best_key && idj < best_id)) {
                    best_key = key;
                    best_id = idj;
                    best = (int32_t)j;
                }
            }
        }
    }
#pragma unroll
    for (int sft = 32; sft > 0; sft >>= 1) {
        const double k2 = __shfl_xor(best_key, sft, 64);
        const uint32_t id2 = (uint32_t)__shfl_xor((int)best_id, sft, 64);
        const int32_t b2 = __shfl_xor(best, sft, 64);
        if (k2 < best_key || (k2 == best_key && id2 < best_id)) {
            best_key = k2;
            best_id = id2;
            best = b2;
        }
    }
    return best;
}

// Wave-aggregated append of this lane's particle to the FP64 recheck list
// (all lanes of the wave must call it).
__device__ __forceinline__ void push_recheck(const Plan& p, uint32_t i, bool need)
{
    const uint64_t mask = __ballot(need);
    if (!mask) return;
    const int lane = threadIdx.x & 63;
    const int leader = __ffsll((unsigned long long)mask) - 1;
    uint32_t base = 0;
    if (lane == leader) base = atomicAdd(&p.ctl->recheck_count, (unsigned int)__popcll(mask));
    base = (uint32_t)__builtin_amdgcn_readlane((int)base, leader);
    if (need) {
        const uint32_t idx = base + (uint32_t)__popcll(mask & ((1ull << lane) - 1ull));
        if (idx < p.recheck_cap) p.recheck[idx] = i;
        else atomicOr(&p.ctl->overflow, 1u);
    }
}

// Full-neighbourhood variant of the search (KMC_SEARCH_FULL): every
// particle scans its own and all 26 neighbouring cells and keeps the running
// (key, id) minimum in registers, writing its partner directly.  It tests
// every pair twice but records nothing, so it suits dense cells with many
// acceptable partners per particle, where the candidate lists of the
// half-neighbourhood search overflow.  Rows and staging as in k_search_half.
// Under the FP32 screen the kept pairs that may still be the best wait in LDS
// (Deferred) and are decided in FP64 after the last row.  One tile of 64 cell-sorted particles (one
// wave), writing their partners; lid: the staged candidates' ids (FP64), dslots:
// the FP32 screen's deferred pairs, both in LDS; STATS: count the pairs for the statistics.
template <class Pol, bool STATS>
__device__ __forceinline__ void search_full_tile(const Plan& p, uint32_t tile, typename Pol::Lds& lds, uint32_t* lid,
                                                 DeferLds* dslots)
{
    const int lane = threadIdx.x;
    const uint32_t i = tile * 64u + (uint32_t)lane;
    const bool valid = i < p.N;
    bool alive = valid && !(p.idB[i] & kGone);   // absorbed particles do not search
    uint32_t bidx = 0, rowkey = 0xFFFFFFFFu;
    int cx = 0, cy = 0, cz = 0;
    typename Pol::Own own{};
    if (alive) {
        bidx = p.boxidx ? p.boxidx[i] : 0u;
        const BoxDev& B = p.boxes[bidx];
        double x, y, z;
        Pol::load_own(lds, p, i, own, x, y, z);
        cx = cell1(x, B.lo[0], B.inv_h[0], B.nc[0]);
        cy = cell1(y, B.lo[1], B.inv_h[1], B.nc[1]);
        cz = cell1(z, B.lo[2], B.inv_h[2], B.nc[2]);
        rowkey = B.coff + (uint32_t)B.nc[0] * ((uint32_t)cy + (uint32_t)B.nc[1] * (uint32_t)cz);
        // adaptive bins: particles in or next to a split cell search their
        // touching leaves instead (k_search_adapt)
        if (p.adapt_L > 0 && p.mixed[rowkey + (uint32_t)cx]) alive = false;
    }
    Best best;
    best.clear();
    Deferred dfr;
    dfr.l = dslots;
    dfr.n = 0;
    uint64_t remaining = __ballot(alive);
    while (remaining) {
        const int lead = __ffsll((unsigned long long)remaining) - 1;
        const uint32_t key = (uint32_t)__builtin_amdgcn_readlane((int)rowkey, lead);
        const int cxf = __builtin_amdgcn_readlane(cx, lead);
        // the row's lanes in ascending cells; a screened group ends after
        // kScreenGroupCells cells (the rest of the row forms the next one),
        // and its span picks its class of screen thresholds
        const uint64_t grp =
            __ballot(alive && rowkey == key && (!Pol::kScreen || cx - cxf < kScreenGroupCells)) & remaining;
        remaining &= ~grp;
        const bool in = (grp >> lane) & 1ull;
        const int last = 63 - __clzll((long long)grp);
        const uint32_t gb = (uint32_t)__builtin_amdgcn_readlane((int)bidx, lead);
        const BoxDev& B = p.boxes[gb];
        const int gcy = __builtin_amdgcn_readlane(cy, lead), gcz = __builtin_amdgcn_readlane(cz, lead);
        const int cxl = __builtin_amdgcn_readlane(cx, last);
        const int NX = B.nc[0], NY = B.nc[1], NZ = B.nc[2];
        typename Pol::Group gctx;
        const uint32_t sbi = gb * (uint32_t)kSpanClasses + span_class(cxl - cxf + 1);
        Pol::begin_group(lds, p, B, own, gctx, cxf, cxl, gcy, gcz, (int)sbi, i, in);
        Pol::group_lds(lds, p, sbi, lane);
        auto part = [&](const auto& m, uint32_t fs, uint32_t fe, uint32_t lf, uint32_t le) {
            for (uint32_t c0 = fs; c0 < fe; c0 += (uint32_t)Pol::W) {
                const uint32_t n = min((uint32_t)Pol::W, fe - c0);
                for (uint32_t t = (uint32_t)lane; t < n; t += 64u) {
                    int wx;
                    const uint32_t j = m.at(c0 + t, wx);
                    Pol::stage(lds, t, p, j, B, gctx, wx, m.wy, m.wz);
                    if constexpr (!Pol::kScreen) lid[t] = p.idB[j];
                }
                __syncthreads();
                const uint32_t f0 = max(lf, c0), f1 = min(le, c0 + n);
                bool shift = false;   // (the screen's records are staged with their image)
                if constexpr (!Pol::kScreen) shift = (m.wx | m.wy | m.wz) != 0;
                if (shift)
                    Pol::template scan_best<true>(lds, lid, c0, f0, f1, i, own, B, gctx, m, best, dfr);
                else
                    Pol::template scan_best<false>(lds, lid, c0, f0, f1, i, own, B, gctx, m, best, dfr);
                __syncthreads();
            }
            // (a particle beyond its slots is searched again: it records nothing
            // more; set in the pair loop this took four registers and with them a wave)
            if (Pol::kScreen && dfr.n > kDefer) best.kcut = -__builtin_inff();
        };
        for (int r = 0; r < 9; ++r) {
            RowRange R;
            int ny = gcy + r % 3 - 1, nz = gcz + r / 3 - 1;
            R.wy = R.wz = 0;
            if (nz < 0) { if (!B.periodic[2]) continue; nz += NZ; R.wz = -1; }
            else if (nz >= NZ) { if (!B.periodic[2]) continue; nz -= NZ; R.wz = 1; }
            if (ny < 0) { if (!B.periodic[1]) continue; ny += NY; R.wy = -1; }
            else if (ny >= NY) { if (!B.periodic[1]) continue; ny -= NY; R.wy = 1; }
            R.row = B.coff + (uint32_t)NX * ((uint32_t)ny + (uint32_t)NY * (uint32_t)nz);
            R.gs = p.start[R.row + (uint32_t)(cxf > 0 ? cxf - 1 : 0)];
            R.ge = p.start[R.row + (uint32_t)(cxl + 1 < NX ? cxl + 1 : NX - 1) + 1u];
            R.ls = R.le = 0u;
            if (in) {
                R.ls = p.start[R.row + (uint32_t)(cx > 0 ? cx - 1 : 0)];
                R.le = p.start[R.row + (uint32_t)(cx + 1 < NX ? cx + 1 : NX - 1) + 1u];
            }
            row_parts<Pol>(p, B, R, true, in, cx, cxf, cxl, part);
        }
    }
    if constexpr (Pol::kScreen) {
        if (alive) Pol::decide_deferred(p, i, dfr, p.boxes[bidx], best);
    }
    if (valid && (alive || p.adapt_L == 0)) p.partner[i] = best.j;
    if (STATS) {
        // statistics: pairs accepted (FP64) or decided in FP64 (FP32 screen)
        uint64_t c = Pol::kScreen ? best.screened : best.accepted;
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) c += __shfl_xor(c, off, 64);
        if (lane == 0 && c) atomicAdd(&p.acc[blockIdx.x % p.acc_lanes].cand, (unsigned long long)c);
    }
    if constexpr (Pol::kScreen) {
        // particles with more deferred pairs than slots
        uint64_t again = __ballot(dfr.n > kDefer);
        if (again) {
            uint32_t own = 0;   // particles in the cell
            if (dfr.n > kDefer && p.N <= kAgainRound) {
                const P64 me = p.B[i];
                const uint32_t c = cell_of(box_of(p, i), me.x, me.y, me.z, false);
                own = p.start[c + 1u] - p.start[c];
            }
            if (__popcll(again) > kAgainAlone || __ballot(own > kAgainCell)) {
                push_recheck(p, i, dfr.n > kDefer);
                again = 0;
            }
        }
        while (again) {
            const int l = __ffsll((unsigned long long)again) - 1;
            again &= again - 1;
            const uint32_t k = tile * 64u + (uint32_t)l;
            const int32_t b = search_one64_wave(p, k);
            if (lane == 0) p.partner[k] = b;
        }
    }
}

template <class Pol>
__global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(Pol::kFullWaves)))
void k_search_full(Plan p)
{
    __shared__ typename Pol::Lds lds;
    if constexpr (Pol::kScreen) {
        __shared__ DeferLds dslots;
        search_full_tile<Pol, true>(p, xcd_tile(blockIdx.x, gridDim.x), lds, nullptr, &dslots);
    } else {
        __shared__ uint32_t lid[Pol::W];
        search_full_tile<Pol, true>(p, xcd_tile(blockIdx.x, gridDim.x), lds, lid, nullptr);
    }
}

// The share of the particles to re-search (one in kRecheckShare) above which the whole-step search is
// the faster way to the same partners (measured on 1e6 particles of one speed,
// three per cell: 1.5 ns a particle re-searched, 0.24 ns a particle of the
// whole step; the crossing is at one in six).
constexpr uint32_t kRecheckShare = 6;
constexpr uint32_t kFallbackBlocks = 4096;

// Whether this step's partners come from the whole-step search: its flag is
// set, or the re-search has too many particles.  (The direct search lists none;
// with the flag set it decides every pair in FP64 itself.)
__device__ __forceinline__ bool whole_step(const Plan& p)
{
    return (p.ctl->overflow != 0u) | (p.ctl->recheck_count > p.N / kRecheckShare + kFallbackBlocks);
}

// Whole-step FP64 search, by the full-neighbourhood organisation, when the
// recheck list overflowed or holds a large share of the particles or, under
// the FP32 screen, a particle lies outside its box's grid or a box's scales
// leave the screen's safe range; otherwise the re-search of the listed
// particles, one wave each.  A fixed grid of waves that exits at once when a
// step needs neither.
template <class Pol>
__global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(Pol::kFullWaves)))
void k_research(Plan p)
{
    __shared__ typename Pol::Lds lds;
    __shared__ uint32_t lid[Pol::W];
    if (!whole_step(p)) {
        const uint32_t n = p.ctl->recheck_count;   // (at most recheck_cap here)
        for (uint32_t k = blockIdx.x; k < n; k += gridDim.x) {
            const uint32_t i = p.recheck[k];
            const int32_t b = search_one64_wave(p, i);
            if (threadIdx.x == 0) p.partner[i] = b;
        }
        return;
    }
    const uint32_t ntiles = (p.N + 63u) / 64u;
    for (uint32_t t = blockIdx.x; t < ntiles; t += gridDim.x) search_full_tile<Pol, false>(p, t, lds, lid, nullptr);
}

// --------------------------------------------------------------------------
// Density-adaptive bins: the search of particles in or next to a split cell.
//
// A particle's candidates are those of the leaves that touch its own, all
// inside the 27 cells around its cell.  A wave takes 64 consecutive sorted
// particles; the sort keeps leaves contiguous, so they fall into a few dozen
// leaves.  For up to kLeafBatch of these at a time kLeafLanes lanes list the
// runs of touching leaves in LDS (a lane takes a neighbour cell, or some rows of
// one where the leaf touches fewer cells than lanes), eight leaves side by
// side.  Then kLeafLanes lanes share a particle and walk its leaf's runs as one
// sequence, each testing every kLeafLanes-th candidate straight from the
// sorted records, one loaded ahead, and their (key, id) minima are folded.
// Each pair is tested from both sides (running minimum, no lists; the order of
// the runs does not matter to the minimum).
//
// Leaves hold few particles (2.5 on average at threshold 8), so it is what a
// wave does per leaf and per candidate besides the test that bounds this: with
// the leaves taken in turn, each listed, staged through LDS and tested by the
// whole wave, half of the instructions and most of the waiting were the listing
// and its barriers.  1e7 particles in blobs, three levels, threshold 8: 4.51 ->
// 2.95 ms; the listing by each particle's lanes for itself 3.57, 4 or 16 lanes
// 3.2 and 3.8, without the load ahead 3.8, a list of a fixed size per leaf 3.25.
// Against the leaves in turn it gains 1.3 to 1.45 times at a threshold of 8 and
// three levels, 1.1 to 1.25 at leaves of 100, and nothing from about 400 on
// (1.0 to 0.89: LDS would serve their many owners better than L1 does).
// Now the L1 lookups of the gathered records and the control flow of the walk
// take about equal parts with the FP64 tests.
// --------------------------------------------------------------------------

// The leaves of the neighbour cell (c + d) that touch the leaf [lo, hi]
// (finest indices per axis) of a particle in cell c, as ranges of the sorted
// arrays: f(s, e) once per run of touching leaves that is contiguous in the
// cell's leaf order (one range for an unsplit cell).  Nothing when the neighbour
// cell does not exist or no leaf of it touches.  For the pair-test counter; the
// search lists a leaf's runs by several lanes (list_leaf).
template <class F>
__device__ __forceinline__ void neighbour_leaves(const Plan& p, const BoxDev& B, const int c[3], const int lo[3],
                                                 const int hi[3], int dx, int dy, int dz, F&& f)
{
    const int L = p.adapt_L;
    const int d[3] = {dx, dy, dz};
    int q[3], w[3];
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        q[a] = c[a] + d[a];
        w[a] = 0;
        if (q[a] < 0) { if (!B.periodic[a]) return; q[a] += B.nc[a]; w[a] = -1; }
        else if (q[a] >= B.nc[a]) { if (!B.periodic[a]) return; q[a] -= B.nc[a]; w[a] = 1; }
    }
    const uint32_t cell = B.coff + (uint32_t)q[0] + (uint32_t)B.nc[0] * ((uint32_t)q[1] + (uint32_t)B.nc[1] * (uint32_t)q[2]);
    const int lvl = (int)p.level[cell];
    const int sh = L - lvl, r = 1 << lvl;
    int jlo[3], jhi[3];
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        // leaf j of the neighbour spans [b0 + j 2^sh, b0 + (j + 1) 2^sh - 1]
        // (b0: its lower face, with the image); it touches [lo, hi] iff
        // (lo - b0 - 1) >> sh <= j <= (hi + 1 - b0) >> sh
        const long long b0 = ((long long)q[a] << L) + (long long)w[a] * ((long long)B.nc[a] << L);
        jlo[a] = (int)max(0ll, ((long long)lo[a] - b0 - 1) >> sh);
        jhi[a] = (int)min((long long)(r - 1), ((long long)hi[a] + 1 - b0) >> sh);
        if (jlo[a] > jhi[a]) return;
    }
    const uint32_t s0 = p.start[cell];
    if (lvl == 0) {
        f(s0, p.start[cell + 1]);
        return;
    }
    const uint32_t* t = p.pool + p.pool_base[cell];
    for (int jz = jlo[2]; jz <= jhi[2]; ++jz)
        for (int jy = jlo[1]; jy <= jhi[1]; ++jy) {
            const uint32_t row = (uint32_t)r * ((uint32_t)jy + (uint32_t)r * (uint32_t)jz);
            f(s0 + t[row + (uint32_t)jlo[0]], s0 + t[row + (uint32_t)jhi[0] + 1u]);
        }
}

// A particle's cell (c) and leaf ([lo, hi] in finest indices) under adaptive
// bins, from its position; returns the linear cell.
__device__ __forceinline__ uint32_t leaf_of(const Plan& p, const BoxDev& B, double x, double y, double z, int c[3],
                                            int lo[3], int hi[3], uint32_t& code)
{
    const int L = p.adapt_L;
    const double xs[3] = {x, y, z};
    int g[3];
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        g[a] = fine1(xs[a], B.lo[a], B.inv_h[a], B.nc[a], L);
        c[a] = g[a] >> L;
    }
    const uint32_t cell = B.coff + (uint32_t)c[0] + (uint32_t)B.nc[0] * ((uint32_t)c[1] + (uint32_t)B.nc[1] * (uint32_t)c[2]);
    const int lvl = (int)p.level[cell];
    const int sh = L - lvl;
    const uint32_t m = (1u << lvl) - 1u;
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        lo[a] = (g[a] >> sh) << sh;
        hi[a] = lo[a] + (1 << sh) - 1;
    }
    code = (((uint32_t)g[0] >> sh) & m) + (m + 1u) * ((((uint32_t)g[1] >> sh) & m) + (m + 1u) * (((uint32_t)g[2] >> sh) & m));
    return cell;
}

constexpr int kLeafLanes = 8;    // lanes that share a leaf's listing, then a particle
constexpr int kLeafBatch = 16;   // leaves listed at a time
// Runs the lists of a batch hold.  One leaf has at most 237: an unsplit cell
// (at most three split levels: 8 x 8 runs from each x face of its neighbours,
// 8 from each y and z face and from the 8 edges along y and z, one from the
// other edges, the corners and the cell itself).
constexpr int kLeafRuns = 256;
static_assert(kLeafRuns >= 237, "one leaf's runs fit");
constexpr uint32_t kNoRun = 0xFFFFFFFFu;

struct AdaptLds {
    int32_t c[64][3];       // per leaf of the wave: its cell,
    uint32_t rl[64];        // ... its place in it (bytes 0 to 2: finest indices of its lower corner; 3: its width)
    uint32_t box[64];
    uint32_t head[kLeafBatch];   // first run of each of the batch's leaves
    uint32_t used;               // runs listed (offered, if more than there is room for)
    uint4 run[kLeafRuns + 1];    // first sorted index, length, image code, the leaf's next run; the last one ends every list
};

// Lists the runs of the leaves that touch leaf l of the wave as entry e of the
// batch; lane u of kLeafLanes.
__device__ __forceinline__ void list_leaf(const Plan& p, const BoxDev& B, AdaptLds& al, uint32_t l, uint32_t e, uint32_t u)
{
    constexpr uint32_t G = (uint32_t)kLeafLanes;
    const int L = p.adapt_L, m = (1 << L) - 1;
    const uint32_t pk = al.rl[l];
    // the range of neighbour cells the leaf touches: three per axis for an
    // unsplit cell, else one or two
    int rl[3], rh[3], d0[3], nd[3];
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        rl[a] = (int)((pk >> (8 * a)) & 0xFFu);
        rh[a] = rl[a] + (int)(pk >> 24) - 1;
        d0[a] = rl[a] == 0 ? -1 : 0;
        nd[a] = (rh[a] == m ? 2 : 1) - d0[a];
    }
    const uint32_t total = (uint32_t)(nd[0] * nd[1] * nd[2]);
    // (a product of ones and twos divides the lanes; 27 cells are taken in turn)
    uint32_t k = u, row0 = 0u, rows = 1u;
    if (total < G) {
        k = u & (total - 1u);
        row0 = u / total;
        rows = G / total;
    }
    // d / n for d < 27 and n of 1, 2, 3
    auto div3 = [](uint32_t d, int n) { return n == 1 ? d : n == 2 ? d >> 1 : (d * 11u) >> 5; };
    for (; k < total; k += G) {
        const uint32_t kxy = div3(k, nd[0]), kz = div3(kxy, nd[1]);
        const int d[3] = {d0[0] + (int)(k - kxy * (uint32_t)nd[0]), d0[1] + (int)(kxy - kz * (uint32_t)nd[1]),
                          d0[2] + (int)kz};
        int q[3], w[3];
        bool ok = true;
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            q[a] = al.c[l][a] + d[a];
            w[a] = q[a] < 0 ? -1 : (q[a] >= B.nc[a] ? 1 : 0);
            if (w[a] != 0) ok = ok && B.periodic[a];
            q[a] -= w[a] * B.nc[a];
        }
        if (!ok) continue;
        const uint32_t cell =
            B.coff + (uint32_t)q[0] + (uint32_t)B.nc[0] * ((uint32_t)q[1] + (uint32_t)B.nc[1] * (uint32_t)q[2]);
        const int lvl = (int)p.level[cell];
        const uint32_t s0 = p.start[cell], s1 = p.start[cell + 1], pb = p.pool_base[cell];
        auto list = [&](uint32_t a, uint32_t b) {
            if (b <= a) return;
            const uint32_t t = atomicAdd(&al.used, 1u);
            if (t >= (uint32_t)kLeafRuns) return;
            al.run[t] = uint4{a, b - a, wcode(w[0], w[1], w[2]), atomicExch(&al.head[e], t)};
        };
        if (lvl == 0) {
            if (row0 == 0u) list(s0, s1);
            continue;
        }
        // the cell's leaves jl .. jh per axis that touch; one run per (y, z)
        const int sh = L - lvl, r = 1 << lvl;
        int jl[3], jh[3];
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            jl[a] = max(0, (rl[a] - (d[a] << L) - 1) >> sh);
            jh[a] = min(r - 1, (rh[a] - (d[a] << L) + 1) >> sh);
        }
        const int ny = jh[1] - jl[1] + 1;
        int jy = jl[1] + (int)row0, jz = jl[2];
        for (;;) {
            while (jy > jh[1]) {
                jy -= ny;
                ++jz;
            }
            if (jz > jh[2]) break;
            const uint32_t* t = p.pool + pb + (uint32_t)r * ((uint32_t)jy + (uint32_t)r * (uint32_t)jz);
            list(s0 + t[jl[0]], s0 + t[jh[0] + 1]);
            jy += (int)rows;
        }
    }
}

template <bool K>
__global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(6))) void k_search_adapt(Plan p)
{
    constexpr uint32_t G = (uint32_t)kLeafLanes;
    __shared__ AdaptLds al;
    const uint32_t lane = threadIdx.x;
    const uint32_t i0 = xcd_tile(blockIdx.x, gridDim.x) * 64u;
    // the wave's particles and their leaves (a leaf's particles are consecutive)
    bool alive = i0 + lane < p.N && !(p.idB[i0 + lane] & kGone);
    uint32_t cell = 0xFFFFFFFFu, code = 0u;
    int c[3] = {0, 0, 0}, lo[3] = {0, 0, 0}, hi[3] = {0, 0, 0};
    uint32_t bidx = 0u;
    if (alive) {
        const P64 me = p.B[i0 + lane];
        bidx = p.boxidx ? p.boxidx[i0 + lane] : 0u;
        cell = leaf_of(p, p.boxes[bidx], me.x, me.y, me.z, c, lo, hi, code);
        alive = p.mixed[cell] != 0;
        if (!alive) cell = 0xFFFFFFFFu;
    }
    const uint32_t cell_l = __shfl_up(cell, 1, 64), code_l = __shfl_up(code, 1, 64);
    const uint64_t lives = __ballot(alive);
    if (lives == 0) return;
    const uint64_t heads = __ballot(alive && (lane == 0u || cell != cell_l || code != code_l));
    const uint32_t nleaves = (uint32_t)__popcll(heads);
    if ((heads >> lane) & 1u) {
        const uint32_t l = (uint32_t)__popcll(heads & ((1ull << lane) - 1ull));
        const int L = p.adapt_L;
        uint32_t pk = (uint32_t)(hi[0] - lo[0] + 1) << 24;
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            al.c[l][a] = c[a];
            pk |= (uint32_t)(lo[a] - (c[a] << L)) << (8 * a);
        }
        al.rl[l] = pk;
        al.box[l] = bidx;
    }
    if (lane == 0u) al.run[kLeafRuns] = uint4{kNoRun, kNoRun, kNoImage, (uint32_t)kLeafRuns};
    const uint32_t u = lane % G, o = lane / G;
    uint32_t accepted = 0u;
    auto search = [&](auto box) {
        uint64_t left = heads;   // heads of the leaves not yet searched
        uint32_t nl = (uint32_t)kLeafBatch;
        for (uint32_t l0 = 0; l0 < nleaves; l0 += nl) {
            nl = min(nl, nleaves - l0);
            if (lane < (uint32_t)kLeafBatch) al.head[lane] = (uint32_t)kLeafRuns;
            if (lane == 0u) al.used = 0u;
            __syncthreads();
            for (uint32_t e = o; e < nl; e += 64u / G) list_leaf(p, box(al.box[l0 + e]), al, l0 + e, e, u);
            __syncthreads();
            if (al.used > (uint32_t)kLeafRuns && nl > 1u) {   // (one leaf always fits)
                __syncthreads();
                nl >>= 1;
                l0 -= nl;
                continue;
            }
            // the particles of these leaves: lanes k0 .. k1 - 1 of the wave
            const uint32_t k0 = (uint32_t)__ffsll((unsigned long long)left) - 1u;
            for (uint32_t e = 0; e < nl; ++e) left &= left - 1ull;
            const uint32_t k1 = left ? (uint32_t)__ffsll((unsigned long long)left) - 1u : 64u;
            for (uint32_t kb = k0; kb < k1; kb += 64u / G) {
                const uint32_t k = kb + o, i = i0 + k;
                const bool on = k < k1 && ((lives >> k) & 1ull);
                if (__ballot(on) == 0) continue;
                Best best;
                best.clear();
                if (on) {
                    const uint32_t l = (uint32_t)__popcll(heads & ((2ull << k) - 1ull)) - 1u, e = l - l0;
                    const P64 me = p.B[i];
                    const BoxDev& B = box(al.box[l]);
                    const uint32_t row = K ? kind_row(p, i) : 0u;
                    const double D2 = B.D2, dt = B.dt;
                    auto test = [&](const P64& q, uint32_t j, uint32_t w) {
                        // (the particle itself has g2 = 0 and is never accepted)
                        double rx = q.x - me.x, ry = q.y - me.y, rz = q.z - me.z;
                        if (w != kNoImage) {
                            const int wx = (int)(w & 3u) - 1, wy = (int)((w >> 2) & 3u) - 1, wz = (int)((w >> 4) & 3u) - 1;
                            if (wx != 0) rx = rx + (double)wx * B.L[0];
                            if (wy != 0) ry = ry + (double)wy * B.L[1];
                            if (wz != 0) rz = rz + (double)wz * B.L[2];
                        }
                        const PairQ pq = pair_q(rx, ry, rz, q.vx - me.vx, q.vy - me.vy, q.vz - me.vz);
                        if (accept(pq, K ? pair_D2(p, B, row, j) : D2, dt)) best.take(pq, p.idB[j], j);
                    };
                    // the run that holds the lane's candidate f
                    uint32_t f = u;
                    uint4 R = al.run[al.head[e]];
                    auto next = [&]() {
                        while (f >= R.y) {
                            f -= R.y;
                            R = al.run[R.w];
                        }
                        return R.x != kNoRun;
                    };
                    if (next()) {
                        P64 q = p.B[R.x + f];
                        for (;;) {
                            const uint32_t j = R.x + f, w = R.z;
                            f += G;
                            if (!next()) {
                                test(q, j, w);
                                break;
                            }
                            const P64 q2 = p.B[R.x + f];
                            test(q, j, w);
                            const uint32_t j2 = R.x + f, w2 = R.z;
                            f += G;
                            const bool more = next();
                            if (more) q = p.B[R.x + f];
                            test(q2, j2, w2);
                            if (!more) break;
                        }
                    }
                }
#pragma unroll
                for (int off = kLeafLanes / 2; off > 0; off >>= 1) {
                    const double k2 = __shfl_xor(best.key, off, 64);
                    const uint32_t id2 = (uint32_t)__shfl_xor((int)best.id, off, 64);
                    const int32_t j2 = __shfl_xor(best.j, off, 64);
                    if (k2 < best.key || (k2 == best.key && id2 < best.id)) {
                        best.key = k2;
                        best.id = id2;
                        best.j = j2;
                    }
                }
                if (on && u == 0u) p.partner[i] = best.j;
                accepted += best.accepted;
            }
            __syncthreads();
        }
    };
    // (one box: its parameters come through scalar loads)
    if (p.boxidx) search([&](uint32_t b) -> const BoxDev& { return p.boxes[b]; });
    else search([&](uint32_t) -> const BoxDev& { return p.boxes[0]; });
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) accepted += __shfl_xor(accepted, off, 64);
    if (lane == 0u && accepted) atomicAdd(&p.acc[blockIdx.x % p.acc_lanes].cand, (unsigned long long)accepted);
}

// --------------------------------------------------------------------------
// Direct search: small gases.
//
// G lanes (a power of two) share a particle and read its candidates straight
// from the sorted records: no staging, no barriers, no lists.  Every lane
// holds the nine row windows of its particle (their starts are loaded
// together) and takes each G-th candidate of every row, the three rows of a z
// plane in flight together; the lanes' (key, id) minima are then folded.  It
// tests every pair from both sides and gives up the reuse of records through
// LDS, so it is for gases that leave the chip idle, where the staged
// searches wait for one row after another (search, list merge and re-search
// together: 4096 particles in 30^3 cells 88 -> 11 us, 1537 at three per cell
// 83 -> 13, 2e4 in the planar mode 25 -> 10, 1e5 at three per cell 57 -> 56).
// FP64: the definition's test.  FP32 screen: FP64 differences rounded to FP32
// against the thresholds of the narrowest groups, which bound larger errors;
// kept pairs are decided in FP64 from the same records.  In a step that breaks
// the screen's assumptions (its flag is set) the screen lets every pair pass.
// --------------------------------------------------------------------------
template <int G, bool K, bool F32>
__global__ __launch_bounds__(64) void k_search_direct(Plan p)
{
    const int lane = threadIdx.x;
    const uint32_t u = (uint32_t)lane % (uint32_t)G;
    const uint32_t i = blockIdx.x * (64u / (uint32_t)G) + (uint32_t)lane / (uint32_t)G;
    const bool alive = i < p.N && !(p.idB[i] & kGone);
    Best best;
    best.clear();
    if (alive) {
        auto search = [&](const BoxDev& B, uint32_t bidx) {
            const P64 me = p.B[i];
            const uint32_t row = K ? kind_row(p, i) : 0u;
            const int NX = B.nc[0], NY = B.nc[1], NZ = B.nc[2];
            const int cx = cell1(me.x, B.lo[0], B.inv_h[0], NX);
            const int cy = cell1(me.y, B.lo[1], B.inv_h[1], NY);
            const int cz = cell1(me.z, B.lo[2], B.inv_h[2], NZ);
            const double D2 = B.D2, dt = B.dt;
            ScreenBounds t{};
            const bool screen = F32 && p.ctl->overflow == 0u;
            if (F32) t = p.box_sb[(size_t)bidx * kSpanClasses];
            auto test = [&](const P64& q, uint32_t j, int wx, int wy, int wz) {
                double rx = q.x - me.x, ry = q.y - me.y, rz = q.z - me.z;
                if (wx != 0) rx = rx + (double)wx * B.L[0];
                if (wy != 0) ry = ry + (double)wy * B.L[1];
                if (wz != 0) rz = rz + (double)wz * B.L[2];
                const double gx = q.vx - me.vx, gy = q.vy - me.vy, gz = q.vz - me.vz;
                if (F32) {
                    const float sx = (float)rx, sy = (float)ry, sz = (float)rz;
                    const float hx = (float)gx, hy = (float)gy, hz = (float)gz;
                    const float b = fmaf(sz, hz, fmaf(sy, hy, sx * hx));
                    const float g2 = fmaf(hz, hz, fmaf(hy, hy, hx * hx));
                    const float rr = fmaf(sz, sz, fmaf(sy, sy, sx * sx));
                    const float kd = K ? p.box_kD2[(size_t)bidx * kSpanClasses * (kMaxKinds * kMaxKinds) + row + p.spB[j]]
                                       : t.kD2;
                    const bool keep = (fmaf(-t.tb1, g2, b) <= t.tb0) & (fmaf(-t.kdt, g2, -b) <= t.tt0) &
                                      (fmaf(rr - kd, g2, -(b * b)) <= t.tc0);
                    if (screen && !keep) return;
                    if (j == i) return;
                    best.screened += 1u;
                }
                const PairQ pq = pair_q(rx, ry, rz, gx, gy, gz);
                // (the particle itself has g2 = 0 and is never accepted)
                if (accept(pq, K ? pair_D2(p, B, row, j) : D2, dt)) best.take(pq, p.idB[j], j);
            };
            // the windows of the nine rows (empty where a row does not exist)
            uint32_t rs[9], re[9];
            int wys[3], wzs[3];
            const int x0 = cx > 0 ? cx - 1 : 0, x1 = cx + 1 < NX ? cx + 1 : NX - 1;
            uint32_t rowbase[9];
            uint32_t exist = 0;
#pragma unroll
            for (int a = 0; a < 3; ++a) {
                int ny = cy + a - 1, nz = cz + a - 1;
                wys[a] = ny < 0 ? -1 : (ny >= NY ? 1 : 0);
                wzs[a] = nz < 0 ? -1 : (nz >= NZ ? 1 : 0);
            }
#pragma unroll
            for (int r = 0; r < 9; ++r) {
                const int wy = wys[r % 3], wz = wzs[r / 3];
                const bool ok = (wy == 0 || B.periodic[1]) && (wz == 0 || B.periodic[2]);
                const int ny = cy + r % 3 - 1 - wy * NY, nz = cz + r / 3 - 1 - wz * NZ;
                rowbase[r] = B.coff + (uint32_t)NX * ((uint32_t)ny + (uint32_t)NY * (uint32_t)nz);
                rs[r] = re[r] = 0u;
                if (ok) {
                    exist |= 1u << r;
                    rs[r] = p.start[rowbase[r] + (uint32_t)x0];
                    re[r] = p.start[rowbase[r] + (uint32_t)x1 + 1u];
                }
            }
#pragma unroll
            for (int z = 0; z < 3; ++z) {
                uint32_t j0 = rs[3 * z] + u, j1 = rs[3 * z + 1] + u, j2 = rs[3 * z + 2] + u;
                const uint32_t e0 = re[3 * z], e1 = re[3 * z + 1], e2 = re[3 * z + 2];
                while (j0 < e0 || j1 < e1 || j2 < e2) {
                    P64 q0, q1, q2;
                    const bool h0 = j0 < e0, h1 = j1 < e1, h2 = j2 < e2;
                    if (h0) q0 = p.B[j0];
                    if (h1) q1 = p.B[j1];
                    if (h2) q2 = p.B[j2];
                    if (h0) test(q0, j0, 0, wys[0], wzs[z]);
                    if (h1) test(q1, j1, 0, wys[1], wzs[z]);
                    if (h2) test(q2, j2, 0, wys[2], wzs[z]);
                    j0 += (uint32_t)G;
                    j1 += (uint32_t)G;
                    j2 += (uint32_t)G;
                }
            }
            if (B.periodic[0] && (cx == 0 || cx == NX - 1)) {
                // the wrapped end cell of every row
                const int wx = cx == 0 ? -1 : 1, c = cx == 0 ? NX - 1 : 0;
                for (int r = 0; r < 9; ++r) {
                    if (!((exist >> r) & 1u)) continue;
                    const int wy = wys[r % 3], wz = wzs[r / 3];
                    const int ny = cy + r % 3 - 1 - wy * NY, nz = cz + r / 3 - 1 - wz * NZ;
                    const uint32_t cell =
                        B.coff + (uint32_t)c + (uint32_t)NX * ((uint32_t)ny + (uint32_t)NY * (uint32_t)nz);
                    const uint32_t e = p.start[cell + 1u];
                    for (uint32_t j = p.start[cell] + u; j < e; j += (uint32_t)G) test(p.B[j], j, wx, wy, wz);
                }
            }
        };
        // (one box: its parameters come through scalar loads)
        if (p.boxidx) {
            const uint32_t b = p.boxidx[i];
            search(p.boxes[b], b);
        } else {
            search(p.boxes[0], 0u);
        }
    }
    uint32_t c = F32 ? best.screened : best.accepted;
#pragma unroll
    for (int off = G / 2; off > 0; off >>= 1) {
        const double k2 = __shfl_xor(best.key, off, 64);
        const uint32_t id2 = (uint32_t)__shfl_xor((int)best.id, off, 64);
        const int32_t j2 = __shfl_xor(best.j, off, 64);
        if (k2 < best.key || (k2 == best.key && id2 < best.id)) {
            best.key = k2;
            best.id = id2;
            best.j = j2;
        }
    }
    if (i < p.N && u == 0) p.partner[i] = best.j;
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) c += __shfl_xor(c, off, 64);
    if (lane == 0 && c) atomicAdd(&p.acc[blockIdx.x % p.acc_lanes].cand, (unsigned long long)c);
}

// Partner of every particle: the (key, id) minimum of its forward best (the
// pairs its own search lane found) and the entries of its candidate list
// (pairs found from the other side, and its own extra pairs); keys are
// exact FP64, ids are read only to break equal keys.  A particle with more
// list entries than slots is searched again in full.
__global__ __launch_bounds__(256) void k_finish(Plan p)
{
    const uint32_t i = blockIdx.x * blockDim.x + threadIdx.x;
    const bool valid = i < p.N;
    const uint32_t cnt = valid ? p.sl_cnt[i] : 0u;
    if (cnt != 0) p.sl_cnt[i] = 0u;
    double best_key = valid ? p.fb_key[i] : 0.0;
    int32_t best = valid ? p.fb_j[i] : -1;
    if (cnt >= 1 && cnt <= (uint32_t)kSlots) {
        for (uint32_t k = 0; k < cnt; ++k) {
            const SlotEntry e = p.sl[(size_t)k * p.N + i];
            const uint32_t j = e.j;
            const double key = e.key;
            // best_key is +inf while there is no best, so an entry with key
            // +inf (a kept pair that the exact test rejected) never wins
            if (key < best_key || (key == best_key && best >= 0 && p.idB[j] < p.idB[best])) {
                best_key = key;
                best = (int32_t)j;
            }
        }
    }
    push_recheck(p, i, cnt > (uint32_t)kSlots);
    if (valid) p.partner[i] = best;
}

// --------------------------------------------------------------------------
// a5-a8: mutual resolve, isotropic CM scatter at t*, free stream, boundary
// conditions, per-step pair count and digest.  One thread per sorted
// particle; both members of a pair compute the pair's update identically and
// each writes only its own particle.
// --------------------------------------------------------------------------

__device__ __forceinline__ void apply_bc(const BoxDev& B, double x[3], double v[3])
{
    if (B.sphere) {
        const double rr = fma(x[2], x[2], fma(x[1], x[1], x[0] * x[0]));
        if (rr > B.R2) {
            const double rn = sqrt(rr);
            const double sc = (2.0 * B.R - rn) / rn;
            const double vn = fma(v[2], x[2], fma(v[1], x[1], v[0] * x[0]));
            const double cf = (2.0 * vn) / rr;
#pragma unroll
            for (int k = 0; k < 3; ++k) {
                v[k] = v[k] - cf * x[k];
                x[k] = x[k] * sc;
            }
        }
        return;
    }
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        const double lo = B.lo[k], hi = B.hi[k];
        if (B.absorb[k]) continue;   // decided by the caller after streaming
        if (B.periodic[k]) {
            if (x[k] >= hi) x[k] = x[k] - B.L[k];
            else if (x[k] < lo) x[k] = x[k] + B.L[k];
        } else {
            if (x[k] < lo) { x[k] = 2.0 * lo - x[k]; v[k] = -v[k]; }
            else if (x[k] > hi) { x[k] = 2.0 * hi - x[k]; v[k] = -v[k]; }
            if (x[k] < lo) x[k] = lo;
            else if (x[k] > hi) x[k] = hi;
        }
    }
}

// Step of sorted particle i: its new record to *out, its id and kind to their
// places, its new position (nx, ny, nz); gone: absorbed earlier or now, left:
// absorbed now; the member of a colliding pair with the smaller id counts the
// collision in my_np and my_dig (all of these are cleared by the caller).
// K: particles of several kinds (masses from the kind table).
template <bool K>
__device__ __forceinline__ void move_particle(const Plan& p, uint32_t i, P64* out, uint64_t& my_np, uint64_t& my_dig,
                                              double& nx, double& ny, double& nz, bool& gone, bool& left)
{
    const BoxDev& B = box_of(p, i);
    const P64 me = p.B[i];
    double x[3] = {me.x, me.y, me.z}, v[3] = {me.vx, me.vy, me.vz};
    uint32_t id = p.idB[i];
    gone = (id & kGone) != 0u;   // absorbed earlier: keeps its state
    const int32_t q = p.partner[i];
    const double dt = B.dt;
    bool hit = false;
    if (q >= 0 && p.partner[q] == (int32_t)i) {
        hit = true;
        const uint32_t idq = p.idB[q];
        const P64 o = p.B[q];
        const double xq[3] = {o.x, o.y, o.z}, vq[3] = {o.vx, o.vy, o.vz};
        const bool me_a = id < idq;   // a = the member with the smaller id
        const double* xa = me_a ? x : xq;
        const double* va = me_a ? v : vq;
        const double* xb = me_a ? xq : x;
        const double* vb = me_a ? vq : v;
        const uint32_t ida = me_a ? id : idq, idb = me_a ? idq : id;
        double r[3], g[3];
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            const int ca = cell1(xa[k], B.lo[k], B.inv_h[k], B.nc[k]);
            const int cb = cell1(xb[k], B.lo[k], B.inv_h[k], B.nc[k]);
            const int w = wrap_of(ca, cb, B.nc[k], B.periodic[k]);
            r[k] = xb[k] - xa[k];
            if (w != 0) r[k] = r[k] + (double)w * B.L[k];
            g[k] = vb[k] - va[k];
        }
        const PairQ pq = pair_q(r[0], r[1], r[2], g[0], g[1], g[2]);
        const double tstar = (-pq.b) / pq.g2;
        double nh[3];
        direction(p.seed, p.ctl->step, ida, nh, p.dims);
        // masses of a and b (particle kinds), equal otherwise
        double ma = 1.0, mb = 1.0;
        if (K) {
            const uint32_t ki = p.spB[i], kq = p.spB[q];
            ma = p.sp_mass[me_a ? ki : kq];
            mb = p.sp_mass[me_a ? kq : ki];
        }
        double vn[3];
        if (ma == mb) {
            const double hg = 0.5 * sqrt(pq.g2);
#pragma unroll
            for (int k = 0; k < 3; ++k) {
                const double vcm = 0.5 * (va[k] + vb[k]);
                vn[k] = me_a ? vcm + hg * nh[k] : vcm - hg * nh[k];
            }
        } else {
            // centre-of-mass velocity, |g| shared in inverse proportion to the masses
            const double M = ma + mb, gm = sqrt(pq.g2);
            const double wa = (mb / M) * gm, wb = (ma / M) * gm;
#pragma unroll
            for (int k = 0; k < 3; ++k) {
                const double vcm = fma(ma, va[k], mb * vb[k]) / M;
                vn[k] = me_a ? vcm + wa * nh[k] : vcm - wb * nh[k];
            }
        }
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            if (p.kinematics == KMC_KIN_AT_TSTAR) {
                const double xs = x[k] + v[k] * tstar;
                x[k] = xs + vn[k] * (dt - tstar);
            } else {
                x[k] = x[k] + vn[k] * dt;
            }
            v[k] = vn[k];
        }
        if (me_a) {
            my_np = 1;
            my_dig = pair_hash(ida, idb);
        }
    }
    if (!hit && !gone) {
#pragma unroll
        for (int k = 0; k < 3; ++k) x[k] = x[k] + v[k] * dt;
    }
    if (!gone) {
        apply_bc(B, x, v);
        // absorbing faces: beyond them the particle leaves the gas
#pragma unroll
        for (int k = 0; k < 3; ++k)
            if (B.absorb[k] && (x[k] < B.lo[k] || x[k] > B.hi[k])) left = true;
        if (left) {
            id |= kGone;
            gone = true;
        }
    }
    P64 w;
    w.x = x[0];
    w.y = x[1];
    w.z = x[2];
    w.vx = v[0];
    w.vy = v[1];
    w.vz = v[2];
    *out = w;
    __builtin_nontemporal_store(id, p.idA + i);
    if (K) p.spA[i] = p.spB[i];
    nx = x[0]; ny = x[1]; nz = x[2];
}

// One kind of particle: compiled for eight waves per SIMD.  The collision
// path is bound by the latency of its partner-record gathers, and the
// default allocation (103 SGPRs) allowed seven; the few scalar values that
// no longer fit go to vector-register lanes (measured 4.36 -> 3.92 ms at
// N = 1e8).  With kinds, eight waves would spill vector registers.
typedef uint32_t Chunk16 __attribute__((ext_vector_type(4), may_alias));   // 16 bytes of a record

template <bool K>
__global__ __launch_bounds__(1024) __attribute__((amdgpu_waves_per_eu(K ? 1 : 8))) void k_resolve(Plan p)
{
    __shared__ uint64_t lds[32];
    extern __shared__ P64 rec[];   // [blockDim.x]: the new records, on their way out
    const uint32_t i = blockIdx.x * blockDim.x + threadIdx.x;
    uint64_t my_np = 0, my_dig = 0;
    double nx = 0.0, ny = 0.0, nz = 0.0;
    bool gone = false, left = false;
    if (i < p.N) move_particle<K>(p, i, rec + threadIdx.x, my_np, my_dig, nx, ny, nz, gone, left);
    // The wave's 64 records leave through LDS, each store instruction writing
    // 1 KiB of consecutive bytes: whole lines, so streaming (non-temporal)
    // stores apply (the state is read again only by the next step's sorted
    // copy).  At 1e8 particles 3.66 ms, against 4.12 with each lane storing its
    // own record and 3.74 with the state in six columns (where the sorted copy,
    // which reads the state back, took 3.43 ms instead of 3.04).
    {
        const uint32_t lane = threadIdx.x & 63u, w0 = threadIdx.x & ~63u;
        const uint32_t i0 = blockIdx.x * blockDim.x + w0;   // the wave's first particle
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
        const Chunk16* src = reinterpret_cast<const Chunk16*>(rec + w0);
        Chunk16* dst = reinterpret_cast<Chunk16*>(p.A + i0);
        const uint32_t nc = i0 < p.N ? 3u * min(64u, p.N - i0) : 0u;
#pragma unroll
        for (uint32_t c = 0; c < 3u; ++c) {
            const uint32_t t = c * 64u + lane;
            if (t < nc) __builtin_nontemporal_store(src[t], dst + t);
        }
    }
    // a1 of the next step: cell and slot of the new position
    bin_particle(p, i, i < p.N, box_of(p, i < p.N ? i : 0u), nx, ny, nz, gone);
    const uint64_t lm = __ballot(left);
    if ((threadIdx.x & 63) == 0 && lm) atomicAdd(&p.ctl->absorbed_total, (unsigned long long)__popcll(lm));
    block_sum2(my_np, my_dig, lds);
    if (threadIdx.x == 0 && my_np != 0) {
        StepAcc& a = p.acc[blockIdx.x % p.acc_lanes];
        atomicAdd(&a.np, (unsigned long long)my_np);
        atomicAdd(&a.dig, (unsigned long long)my_dig);
    }
}

// End of step (one block): fold this step's partial sums into its history row
// and the running candidate count, clear them, and advance the boxes' time
// and the step counters.
__global__ __launch_bounds__(1024) void k_advance(Plan p)
{
    __shared__ uint64_t lds[32];
    uint64_t np = 0, dig = 0, cand = 0, z = 0;
    const bool whole = whole_step(p);   // (loaded here, under the sums)
    for (uint32_t k = threadIdx.x; k < p.acc_lanes; k += blockDim.x) {
        StepAcc& a = p.acc[k];
        np += a.np;
        dig += a.dig;
        cand += a.cand;
        a.np = 0;
        a.dig = 0;
        a.cand = 0;
    }
    for (uint32_t b = threadIdx.x; b < p.nboxes; b += blockDim.x) p.boxes[b].time = p.boxes[b].time + p.boxes[b].dt;
    block_sum2(np, dig, lds);
    __syncthreads();
    block_sum2(cand, z, lds);
    if (threadIdx.x == 0) {
        const unsigned long long done = p.ctl->steps_done;
        p.hist_np[done % p.H] = np;
        p.hist_dig[done % p.H] = dig;
        p.ctl->candidates_total += cand;
        p.ctl->rechecks_total += p.ctl->recheck_count;
        p.ctl->fallbacks_total += whole ? 1ull : 0ull;
        p.ctl->steps_done = done + 1;
        p.ctl->step += 1;
    }
}

// Pair tests of the last step: sum over sorted particles of the 27-cell
// neighbourhood population minus one.
__global__ __launch_bounds__(256) void k_count_tests(Plan p, unsigned long long* out)
{
    __shared__ uint64_t lds[32];
    const uint32_t i = blockIdx.x * blockDim.x + threadIdx.x;
    uint64_t t = 0, z = 0;
    if (i < p.N && !(p.idB[i] & kGone)) {
        const BoxDev& B = box_of(p, i);
        const P64 me = p.B[i];
        const int cx = cell1(me.x, B.lo[0], B.inv_h[0], B.nc[0]);
        const int cy = cell1(me.y, B.lo[1], B.inv_h[1], B.nc[1]);
        const int cz = cell1(me.z, B.lo[2], B.inv_h[2], B.nc[2]);
        const uint32_t cell = B.coff + (uint32_t)cx + (uint32_t)B.nc[0] * ((uint32_t)cy + (uint32_t)B.nc[1] * (uint32_t)cz);
        if (p.adapt_L > 0 && p.mixed[cell]) {
            // adaptive bins: the particles of the touching leaves
            int c[3], lo[3], hi[3];
            uint32_t code;
            leaf_of(p, B, me.x, me.y, me.z, c, lo, hi, code);
            for (int k = 0; k < 27; ++k)
                neighbour_leaves(p, B, c, lo, hi, k % 3 - 1, (k / 3) % 3 - 1, k / 9 - 1,
                                 [&](uint32_t s, uint32_t e) { t += e - s; });
        } else {
            for_each_range(B, cx, cy, cz, p.start, [&](uint32_t s, uint32_t e, int, int, int) { t += e - s; });
        }
        t -= 1;
    }
    block_sum2(t, z, lds);
    if (threadIdx.x == 0) atomicAdd(out, (unsigned long long)t);
}

// Candidates of all particles of the initial state, from the cell counts of
// its binning (before the first step's scan clears them).
__global__ __launch_bounds__(256) void k_init_tests(Plan p)
{
    __shared__ uint64_t lds[32];
    const uint32_t i = blockIdx.x * blockDim.x + threadIdx.x;
    uint64_t t = 0, z = 0;
    if (i < p.N) {
        const BoxDev& B = box_of(p, i);
        const P64 me = p.A[i];
        const double xs[3] = {me.x, me.y, me.z};
        int c[3];
#pragma unroll
        for (int a = 0; a < 3; ++a) c[a] = cell1(xs[a], B.lo[a], B.inv_h[a], B.nc[a]);
        for (int k = 0; k < 27; ++k) {
            const int d[3] = {k % 3 - 1, (k / 3) % 3 - 1, k / 9 - 1};
            int q[3];
            bool ok = true;
#pragma unroll
            for (int a = 0; a < 3; ++a) {
                q[a] = c[a] + d[a];
                if (q[a] < 0) { ok = ok && B.periodic[a]; q[a] += B.nc[a]; }
                else if (q[a] >= B.nc[a]) { ok = ok && B.periodic[a]; q[a] -= B.nc[a]; }
            }
            if (ok)
                t += p.count[B.coff + (uint32_t)q[0] +
                             (uint32_t)B.nc[0] * ((uint32_t)q[1] + (uint32_t)B.nc[1] * (uint32_t)q[2])];
        }
    }
    block_sum2(t, z, lds);
    if (threadIdx.x == 0) atomicAdd(&p.ctl->tests_init, (unsigned long long)t);
}

// Waves that walk the list of split cells (adaptive bins).
constexpr uint32_t kAdaptPrepBlocks = 4096;

inline uint32_t blocks_for(uint32_t n, uint32_t b) { return (n + b - 1) / b; }

// The direct search with G lanes per particle.
template <int G>
void launch_direct(hipStream_t s, const Plan& p)
{
    const uint32_t g = blocks_for(p.N, 64 / G);
    const bool f32 = p.precision == KMC_FP32_SCREEN;
    if (p.nspecies > 0) {
        if (f32) k_search_direct<G, true, true><<<g, 64, 0, s>>>(p);
        else k_search_direct<G, true, false><<<g, 64, 0, s>>>(p);
    } else {
        if (f32) k_search_direct<G, false, true><<<g, 64, 0, s>>>(p);
        else k_search_direct<G, false, false><<<g, 64, 0, s>>>(p);
    }
}

// The search kernel of one precision policy and tile shape.
template <template <bool, class> class Pol, class T>
void launch_search(bool kinds, bool full, uint32_t gW, hipStream_t s, const Plan& p)
{
    if (full) {
        if (kinds) k_search_full<Pol<true, T>><<<gW, 64, 0, s>>>(p);
        else k_search_full<Pol<false, T>><<<gW, 64, 0, s>>>(p);
    } else {
        if (kinds) k_search_half<Pol<true, T>><<<gW, 64, 0, s>>>(p);
        else k_search_half<Pol<false, T>><<<gW, 64, 0, s>>>(p);
    }
}

}  // namespace

// --------------------------------------------------------------------------
// Launchers
// --------------------------------------------------------------------------

hipError_t launch_init(const Plan& p, const double* d_state, const uint8_t* d_kind, hipStream_t s)
{
    const uint32_t b = 256;
    if (p.N > 0) k_init_particles<<<blocks_for(p.N, b), b, 0, s>>>(p, d_state, d_kind);
    k_fill_u32<<<blocks_for(p.C, b) < 4096 ? blocks_for(p.C, b) : 4096, b, 0, s>>>(p.count, p.C, 0u);
    if (p.N > 0) k_fill_u32<<<4096, b, 0, s>>>(p.sl_cnt, (size_t)p.N, 0u);
    k_init_ctl<<<1, 64, 0, s>>>(p, 0);
    if (p.N > 0 && p.nspecies > 0) k_check_kinds<<<blocks_for(p.N, b), b, 0, s>>>(p, d_kind);
    if (p.N > 0) k_bin<<<blocks_for(p.N, b), b, 0, s>>>(p);
    return hipGetLastError();
}

hipError_t launch_init_tests(const Plan& p, hipStream_t s)
{
    if (p.N > 0) k_init_tests<<<blocks_for(p.N, 256), 256, 0, s>>>(p);
    return hipGetLastError();
}

hipError_t launch_step(const Plan& p, hipStream_t s, hipEvent_t* ev)
{
    const uint32_t b = (uint32_t)p.block;
    const uint32_t gN = blocks_for(p.N, b);
    auto mark = [&](int k) { if (ev) (void)hipEventRecord(ev[k], s); };
    mark(KMC_PHASE_BIN);   // binning runs at the end of the previous step (k_resolve) or in kmc_init
    mark(KMC_PHASE_SCAN);
    if (p.C <= kOneScanCells && p.adapt_L == 0) {
        k_scan_one<<<1, 1024, 0, s>>>(p);
    } else {
        k_scan_reduce<<<p.nblk_scan, p.scan_block, 0, s>>>(p);
        if (p.nblk_scan <= kSumBlocks) {
            k_scan_down<true><<<p.nblk_scan, p.scan_block, 0, s>>>(p);
        } else {
            k_scan_partials<<<1, 1024, 0, s>>>(p);
            k_scan_down<false><<<p.nblk_scan, p.scan_block, 0, s>>>(p);
        }
    }
    if (p.adapt_L > 0 && p.N > 0) {
        // adaptive bins: split cells' leaf tables, then every particle's rank in its leaf
        k_refined_prep<<<kAdaptPrepBlocks, 64, 0, s>>>(p);
        k_leaf_count<<<gN, b, 0, s>>>(p);
        k_leaf_scan<<<kAdaptPrepBlocks, 64, 0, s>>>(p);
    }
    mark(KMC_PHASE_SCATTER);
    if (p.N > 0) {
        if (p.precision == KMC_FP32_SCREEN) k_scatter<true><<<gN, b, 0, s>>>(p);
        else k_scatter<false><<<gN, b, 0, s>>>(p);
    }
    const uint32_t gW = blocks_for(p.N, 64);
    if (p.precision == KMC_FP32_SCREEN || p.dt_rule == KMC_DT_ADAPTIVE) {
        if (p.nblk_part <= kFoldAlone) {
            k_step_setup<true><<<p.nboxes, 64 * kSpanClasses, 0, s>>>(p);
        } else {
            k_fold_partials<<<p.nboxes * kVmaxSplit, 256, 0, s>>>(p);
            k_step_setup<false><<<p.nboxes, 64 * kSpanClasses, 0, s>>>(p);
        }
    }
    mark(KMC_PHASE_SEARCH);
    if (ev) (void)hipEventRecord(ev[KMC_PHASE_COUNT + 1], s);   // search kernel alone
    const int32_t dg = p.direct;
    const bool full = p.search_mode == KMC_SEARCH_FULL || dg > 0;
    if (dg > 0) {
        if (dg == 4) launch_direct<4>(s, p);
        else if (dg == 8) launch_direct<8>(s, p);
        else launch_direct<16>(s, p);
    } else if (p.N > 0) {
        const bool kinds = p.nspecies > 0;
        if (p.precision == KMC_FP32_SCREEN) {
            if (p.tile == 1) launch_search<PolF32, TileF32_1>(kinds, full, gW, s, p);
            else if (p.tile == 2) launch_search<PolF32, TileF32_2>(kinds, full, gW, s, p);
            else launch_search<PolF32, TileF32_0>(kinds, full, gW, s, p);
        } else {
            if (p.tile == 1) launch_search<PolF64, TileF64_1>(kinds, full, gW, s, p);
            else if (p.tile == 2) launch_search<PolF64, TileF64_2>(kinds, full, gW, s, p);
            else launch_search<PolF64, TileF64_0>(kinds, full, gW, s, p);
        }
    }
    if (p.N > 0 && p.adapt_L > 0) {
        // the particles next to split cells: plain FP64 in both precisions
        // (their groups are leaves of a few particles, where the screen's
        // conversions and FP64 decisions cost more than they save)
        if (p.nspecies > 0) k_search_adapt<true><<<gW, 64, 0, s>>>(p);
        else k_search_adapt<false><<<gW, 64, 0, s>>>(p);
    }
    mark(KMC_PHASE_FINISH);
    if (p.N > 0 && !full) {
        k_finish<<<blocks_for(p.N, 256), 256, 0, s>>>(p);
    }
    mark(KMC_PHASE_RECHECK);
    // (in FP64 the full search lists nothing; under the FP32 screen it may, and
    // the sorted copy may ask for the whole-step search)
    if (p.N > 0 && dg == 0 && (!full || p.precision == KMC_FP32_SCREEN)) {
        const uint32_t g = gW < kFallbackBlocks ? gW : kFallbackBlocks;
        if (p.nspecies > 0) k_research<PolF64<true>><<<g, 64, 0, s>>>(p);
        else k_research<PolF64<false>><<<g, 64, 0, s>>>(p);
    }
    mark(KMC_PHASE_RESOLVE);
    if (p.N > 0) {
        if (p.nspecies > 0) k_resolve<true><<<gN, b, b * sizeof(P64), s>>>(p);
        else k_resolve<false><<<gN, b, b * sizeof(P64), s>>>(p);
    }
    k_advance<<<1, p.acc_lanes, 0, s>>>(p);
    mark(KMC_PHASE_COUNT);
    return hipGetLastError();
}

hipError_t launch_read_partners(const Plan& p, int32_t* out, hipStream_t s)
{
    if (p.N > 0) k_read_partners<<<blocks_for(p.N, 256), 256, 0, s>>>(p, out);
    return hipGetLastError();
}

// Above this size the state is read out by the gather (two launches): direct
// 4.1 us against 4.9 at 3e4 particles, 8.0 against 5.8 at 1e5, 76 against 42
// at 1e6.
constexpr uint32_t kStateGatherMin = 65536;

hipError_t launch_read_state(const Plan& p, double* out, hipStream_t s)
{
    if (p.N > kStateGatherMin) {
        k_state_places<<<blocks_for(p.N, 256), 256, 0, s>>>(p);
        k_state_gather<<<blocks_for(p.N, 256), 256, 0, s>>>(p, out);
    } else if (p.N > 0) {
        k_read_state<<<blocks_for(p.N, 256), 256, 0, s>>>(p, out);
    }
    return hipGetLastError();
}

hipError_t launch_count_tests(const Plan& p, unsigned long long* d_out, hipStream_t s)
{
    if (p.N > 0) k_count_tests<<<blocks_for(p.N, 256), 256, 0, s>>>(p, d_out);
    return hipGetLastError();
}

}  // namespace kmc
