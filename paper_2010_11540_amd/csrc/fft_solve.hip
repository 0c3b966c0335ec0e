// Grid-side kernels of libscpic for gfx950: the exact reduction of the
// per-workgroup charge partials and the open-boundary Poisson solve as a
// zero-padded FFT convolution with the free-space Green's function (Hockney's
// method), the centred-difference field taken in the spectrum.  Each axis is
// padded to the power of two mx >= 2 nx (my >= 2 ny): any such length makes
// the cyclic convolution equal the linear one on nodes -1..n.  Hand-written
// radix-4/2 Stockham FFTs in registers, each run by (part of) one wave, their
// exchanges between stages through XOR-swizzled LDS buffers on which no
// stage's accesses conflict; no vendor FFT library.
//
// Data flow for a charge grid q (nx x ny, rows i along x; hy = my / 2):
//   k_rows_fwd   one workgroup per row i: sum the row's partials exactly
//                (uint64, + carries) or read a dense int64 row, scale to
//                rho; the real row zero-padded to my is transformed as a
//                complex FFT of half length hy (even/odd samples packed) and
//                untangled into the half spectrum l = 0..hy   -> A^T [hy+1][nx]
//   k_cols       per column l: FFT along x (length mx, zero-padded),
//                multiply by the real Green's spectrum G^(k,l) (inverse-FFT
//                normalisation folded in), then two inverse FFTs run by two
//                groups of lanes: -i sin(2 pi k/mx)/dx * Phi (the x central
//                difference) and Phi, scaled by -i sin(2 pi l/my)/dy (the y
//                central difference); rows 0..nx-1 kept -> (Bx, By) [nx][hy+1]
//   k_rows_inv   per row i: both half spectra packed as Ex + i Ey, completed
//                by Hermitian symmetry, one inverse FFT     -> ex, ey [nx][ny]
// Taking the differences in the spectrum keeps the large constant part of
// the potential out of the field's rounding, which matters for the FP32 form.
// The column and row-inverse kernels issue all of their global loads into
// registers before their first transform and so wait for one round of memory
// latency; the row kernel for two per kReduceChunk partial slices of a lane (the
// headers, then the slices).
#include <algorithm>
#include <type_traits>

#include "scpic_internal.h"

// The solve fuses the multiply-adds it names (twiddle) and no others, so the
// batched and the single-beam kernels, whose lengths are compiled apart, give
// the same bits.
#pragma clang fp contract(off)

namespace scpic {
namespace {

template <typename T>
struct cx {
    T re, im;
};

template <typename T>
__device__ __forceinline__ cx<T> operator+(cx<T> a, cx<T> b) { return {a.re + b.re, a.im + b.im}; }
template <typename T>
__device__ __forceinline__ cx<T> operator-(cx<T> a, cx<T> b) { return {a.re - b.re, a.im - b.im}; }
// d * w with each part one product and one fused multiply-add
template <typename T>
__device__ __forceinline__ cx<T> twiddle(cx<T> d, cx<T> w)
{
    return {fma(d.re, w.re, -(d.im * w.im)), fma(d.im, w.re, d.re * w.im)};
}
template <typename T>
__device__ __forceinline__ cx<T> conj(cx<T> a) { return {a.re, -a.im}; }
template <typename T>
__device__ __forceinline__ cx<T> scale_c(cx<T> a, T s) { return {a.re * s, a.im * s}; }
// -i * a
template <typename T>
__device__ __forceinline__ cx<T> mul_neg_i(cx<T> a) { return {a.im, -a.re}; }
// +i * a
template <typename T>
__device__ __forceinline__ cx<T> mul_pos_i(cx<T> a) { return {-a.im, a.re}; }

// Orders one wave's LDS accesses across an FFT stage: a wave's LDS
// instructions execute in order, so the fences only stop the compiler from
// moving a read of the next stage above a write of this one.
__device__ __forceinline__ void wave_lds_order()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// LDS slot of element e of an FFT buffer: e with bits 0-4 XORed by bits 2-6
// (a permutation within each aligned block of 32 elements, and of any
// shorter buffer).  With it the strided writes of the early FFT stages (and
// their reads) fall on distinct banks, which the natural order does not:
// there a stage's outputs are written 4 ns elements apart per lane.
__device__ __forceinline__ int sw(int e) { return e ^ ((e >> 2) & 31); }

// Forward DFT X[k] = sum_n x[n] exp(-2 pi i n k / L), L = 2^LOG2, of a
// sequence held in registers by a group of G lanes of one wave, E elements
// per lane: lane t (0 <= t < G) holds element t + G r in v[r], before and
// after.  Stockham autosort: radix-4 stages after one radix-2 stage when LOG2
// is odd; the first stage reads and the last one writes the lane's own
// elements, and only the exchanges between stages go through LDS (buf: L
// elements of the group's own).  One wave's LDS accesses execute in order, so
// a transform needs no barrier and no second buffer.  Every stage multiplies
// by the entries of the stage twiddle table (stage_twiddle_count), which each
// lane loads into registers once for all its transforms.
//
// A transform is a chain of latencies, not of work: of the ~1 us a 256-point
// FP64 transform took with every stage reading and writing LDS, most was the
// round trip of each stage and its twiddle reads.  Held in registers, a
// forward transform, the product with the Green's spectrum and an inverse
// make 6 exchanges instead of 12 and need no barrier between them.  Per
// space-charge step, FP64: 1e6 particles on 128^2 34.5 -> 31.9 us, 1e4 on 64^2
// 19.4 -> 16.9 us, the 64-beam scan 235 -> 222 us (its column kernel 26 -> 17
// us, row-inverse 12 -> 8 us: a wave's lanes all transform, where one wave of
// four did), the same bits.
//
// 4 elements per lane (one butterfly) leave a stage's work at its least;
// L = 512 takes 8, which 64 lanes need, and there the radix-2 stage and the
// first radix-4 stage share the lane's elements (no exchange between them).
// With 8 per lane for every odd LOG2 the 128-point transforms, one exchange
// shorter but twice the instructions per stage, were no faster than in LDS.
template <typename T, int LOG2>
struct WaveFft {
    static constexpr int L = 1 << LOG2;
    static constexpr int E = LOG2 == 9 ? 8 : 4;
    static constexpr int G = L / E;              // lanes of one transform
    static constexpr int B = E / 4;              // radix-4 butterflies per lane and stage
    static constexpr int C = (LOG2 & 1) ? 2 : 1;  // ns of the first radix-4 stage
    static constexpr int kStages = LOG2 / 2;     // radix-4 stages
    static constexpr bool kPre = C == 2 && E == 4;  // radix-2 stage with an exchange of its own
    static constexpr int kDone = kPre ? 0 : 1;   // radix-4 stages before the first exchange
    static_assert(G >= 1 && G <= 64, "a transform lives in one wave");

    cx<T> w[kStages - kDone][B][3];  // of the stages after the first exchange
    cx<T> w0[E == 8 ? 3 : 1];        // first radix-4 stage's k = 1 (E == 8)

    __device__ __forceinline__ void load(const cx<T> *__restrict__ st, int t)
    {
        if constexpr (E == 8)
#pragma unroll
            for (int m = 0; m < 3; ++m) w0[m] = st[3 + m];
        int ns = kDone ? 4 * C : C;
#pragma unroll
        for (int s = 0; s + kDone < kStages; ++s, ns *= 4)
#pragma unroll
            for (int b = 0; b < B; ++b) {
                const int k = (t + G * b) & (ns - 1);
#pragma unroll
                for (int m = 0; m < 3; ++m) w[s][b][m] = st[ns - C + 3 * k + m];
            }
    }

    static __device__ __forceinline__ void butterfly(cx<T> &a0, cx<T> &a1, cx<T> &a2, cx<T> &a3)
    {
        const cx<T> t0 = a0 + a2, t1 = a0 - a2, t2 = a1 + a3, t3 = a1 - a3;
        a0 = t0 + t2;
        a1 = t1 + mul_neg_i(t3);
        a2 = t0 - t2;
        a3 = t1 + mul_pos_i(t3);
    }

    __device__ __forceinline__ void run(cx<T> (&v)[E], cx<T> *buf, int t) const
    {
        // the stages before the first exchange, on the lane's own elements
        if constexpr (E == 8) {
            cx<T> p[4], q[4];
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                p[r] = v[r] + v[r + 4];
                q[r] = v[r] - v[r + 4];
            }
            // radix-4 butterflies 2 t (k = 0) and 2 t + 1 (k = 1); together
            // their outputs are elements 8 t .. 8 t + 7
            butterfly(p[0], p[1], p[2], p[3]);
#pragma unroll
            for (int m = 0; m < 3; ++m) q[m + 1] = twiddle(q[m + 1], w0[m]);
            butterfly(q[0], q[1], q[2], q[3]);
#pragma unroll
            for (int m = 0; m < 4; ++m) {
                buf[sw(8 * t + 2 * m)] = p[m];
                buf[sw(8 * t + 2 * m + 1)] = q[m];
            }
        } else if constexpr (kPre) {
#pragma unroll
            for (int r = 0; r < 2; ++r) {
                const int e = 2 * (t + G * r);
                buf[sw(e)] = v[r] + v[r + 2];
                buf[sw(e + 1)] = v[r] - v[r + 2];
            }
        } else {
            butterfly(v[0], v[1], v[2], v[3]);
#pragma unroll
            for (int r = 0; r < 4; ++r) buf[sw(4 * t + r)] = v[r];
        }
        int ns = kDone ? 4 * C : C;
#pragma unroll
        for (int s = 0; s + kDone < kStages; ++s, ns *= 4) {
            wave_lds_order();
#pragma unroll
            for (int r = 0; r < E; ++r) v[r] = buf[sw(t + G * r)];
#pragma unroll
            for (int b = 0; b < B; ++b) {
                // butterfly j = t + G b reads elements j + m L / 4 = t + G (b + B m)
#pragma unroll
                for (int m = 1; m < 4; ++m) v[b + B * m] = twiddle(v[b + B * m], w[s][b][m - 1]);
                butterfly(v[b], v[b + B], v[b + 2 * B], v[b + 3 * B]);
            }
            if (s + kDone + 1 < kStages) {
                wave_lds_order();
#pragma unroll
                for (int b = 0; b < B; ++b) {
                    const int j = t + G * b, k = j & (ns - 1), base = (j - k) * 4 + k;
#pragma unroll
                    for (int m = 0; m < 4; ++m) buf[sw(base + m * ns)] = v[b + B * m];
                }
            }
        }
        // the last stage's output j + m L / 4 is element t + G (b + B m): the
        // lane's own again.  The next transform may use buf at once.
        wave_lds_order();
    }
};

// Calls f(std::integral_constant<int, log2>), LO <= log2 <= HI.
template <int LO, int HI, typename F>
__host__ __device__ __forceinline__ void with_log2(int log2, F &&f)
{
    if constexpr (LO < HI) {
        if (log2 == LO)
            f(std::integral_constant<int, LO>{});
        else
            with_log2<LO + 1, HI>(log2, f);
    } else {
        f(std::integral_constant<int, HI>{});
    }
}

constexpr int kRowThreads = 1024;   // row-forward: 16 waves share the reduction
constexpr int kLineThreads = 256;   // batched column and row-inverse kernels

// Exact sum of grid row i over the partials of nblocks workgroups plus the
// carry grid (which is cleared), for the ny cells of the row.  Called by all
// NT threads of the workgroup (NT >= ny).  Thread t reads 16-byte chunks (4 cells) of the row:
// ny/4 lanes cover one workgroup's row segment and the NT/(ny/4) groups of
// lanes split the workgroups.  Each lane reads the headers of its workgroups
// itself (a group's lanes the same ones), then issues kReduceChunk chunk loads
// before adding any: two rounds of memory latency for kReduceChunk workgroups
// per lane, and no barrier between them.  Chunks outside a
// workgroup's bounding box are not read (their loads return zeros without
// touching memory).  red: LDS scratch of NT * 4 uint64; carry_v: this cell's
// carry, loaded by the caller with its first round of loads (cleared here
// when nonzero).  Returns the total of cell tid (tid < ny).
// Four at a time is the faster also where a lane has more workgroups (with 256
// pass workgroups 4 at ny = 64, 8 at 128, 16 at 256) and so twice the rounds.
// Row kernel, us, four and eight: 1e4 particles on 64^2 4.4, 5.0; 1e6 on 64^2 4.9,
// 5.8; on 128^2 6.4, 6.6; on 176^2 7.7, 8.8; on 256^2 10.0, 11.0.  Eight only where
// a lane has more than four: 6.6 on 128^2, 8.7 on 176^2, 10.9 on 256^2.
constexpr int kReduceChunk = 4;

// Lane layout of a row reduction by NT threads: lanes = ny/4 16-byte chunks
// cover one workgroup's row segment (ny is a multiple of 4), and groups =
// NT/lanes whole groups of lanes split the workgroups.
struct RowLanes {
    int lanes, groups, grp, j0c;
};
template <int NT>
__device__ __forceinline__ RowLanes row_lanes(int ny, int tid)
{
    RowLanes r;
    r.lanes = ny >> 2;
    r.groups = NT / r.lanes;  // ny <= 256 -> at least NT / 64
    r.grp = tid / r.lanes;
    r.j0c = (tid - r.grp * r.lanes) * 4;
    return r;
}

template <int NT>
__device__ __forceinline__ unsigned long long reduce_row(const DepositTarget &dep,
                                                         unsigned long long *red, int nblocks,
                                                         int i, int ny, int tid,
                                                         unsigned long long carry_v)
{
    const RowLanes L = row_lanes<NT>(ny, tid);
    const int groups = L.groups, grp = L.grp, j0c = L.j0c;
    // when ny / 4 does not divide NT the last threads form no whole group
    const bool member = grp < groups;
    // The partials as a buffer: a chunk outside a workgroup's box is read at
    // an offset past the buffer's end, which returns zeros and touches no
    // memory.  A chunk inside the box holds the box's cells and zeros (the
    // tile's cells outside the box are zero), so no cell needs a mask.
    const uint32_t bytes = (uint32_t)(sizeof(uint32_t) * (size_t)dep.max_blocks * ny) *
                           (uint32_t)(i + 1);
    const __amdgpu_buffer_rsrc_t rs =
        __builtin_amdgcn_make_buffer_rsrc(dep.partial, (short)0, (int)bytes, 0x00020000);
    constexpr uint32_t kOutside = 0x80000000u;
    const uint32_t row0 = (uint32_t)(sizeof(uint32_t) * ((size_t)i * dep.max_blocks * ny + j0c));
    unsigned long long s0 = 0, s1 = 0, s2 = 0, s3 = 0;
    for (int b0 = member ? grp : nblocks; b0 < nblocks; b0 += groups * kReduceChunk) {
        uint2 box[kReduceChunk];  // rows, cols of the header
#pragma unroll
        for (int u = 0; u < kReduceChunk; ++u) {
            const int b = b0 + u * groups;
            box[u] = *reinterpret_cast<const uint2 *>(&dep.header[b < nblocks ? b : 0].rows);
        }
        uint32_t off[kReduceChunk];
#pragma unroll
        for (int u = 0; u < kReduceChunk; ++u) {
            const int b = b0 + u * groups;
            const bool take = b < nblocks && i >= (int)(box[u].x & 0xffffu) &&
                              i <= (int)(box[u].x >> 16) &&
                              j0c + 3 >= (int)(box[u].y & 0xffffu) && j0c <= (int)(box[u].y >> 16);
            off[u] = take ? row0 + (uint32_t)(sizeof(uint32_t) * (size_t)b * ny) : kOutside;
        }
        // every load in flight before the first add
        decltype(__builtin_amdgcn_raw_buffer_load_b128(rs, 0, 0, 0)) v[kReduceChunk];
#pragma unroll
        for (int u = 0; u < kReduceChunk; ++u)
            v[u] = __builtin_amdgcn_raw_buffer_load_b128(rs, (int)off[u], 0, 0);
#pragma unroll
        for (int u = 0; u < kReduceChunk; ++u) {
            s0 += (uint32_t)v[u][0];
            s1 += (uint32_t)v[u][1];
            s2 += (uint32_t)v[u][2];
            s3 += (uint32_t)v[u][3];
        }
    }
    if (member) {
        unsigned long long *mine = red + (size_t)grp * ny + j0c;
        mine[0] = s0;
        mine[1] = s1;
        mine[2] = s2;
        mine[3] = s3;
    }
    __syncthreads();
    unsigned long long t = 0;
    if (tid < ny) {
#pragma unroll 8
        for (int g = 0; g < groups; ++g) t += red[(size_t)g * ny + tid];
        t += carry_v;
        if (carry_v) dep.carry[(size_t)i * ny + tid] = 0ull;
    }
    return t;
}

// Exact int64 charge grid (scpic_deposit): one workgroup per row.
__global__ void __launch_bounds__(kRowThreads)
    k_reduce(DepositTarget dep, int nblocks, int nx, int ny, int64_t *__restrict__ q,
             int64_t *__restrict__ n_in)
{
    __shared__ unsigned long long red[kRowThreads * 4];
    const int tid = threadIdx.x, i = blockIdx.x;
    const unsigned long long cv = tid < ny ? dep.carry[(size_t)i * ny + tid] : 0ull;
    const unsigned long long t = reduce_row<kRowThreads>(dep, red, nblocks, i, ny, tid, cv);
    if (tid < ny) q[(size_t)i * ny + tid] = (int64_t)t;
    if (n_in != nullptr && i == 0 && tid < 64) {
        long long cnt = 0;
        for (int b = tid; b < nblocks; b += 64) cnt += dep.header[b].count;
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) cnt += __shfl_xor(cnt, o, 64);
        if (tid == 0) *n_in = cnt;
    }
}

// Row i of rho (from the partials when FROM_PARTIALS, else from a dense int64
// grid), real and zero-padded to my = 2 hy: packed z[m] = rho[2m] + i rho[2m+1]
// (zero from index ny on), Z = FFT_hy(z), then
//   X[l] = (Z[l] + conj Z[hy-l]) / 2 - i W^l (Z[l] - conj Z[hy-l]) / 2,
// W = exp(-2 pi i / my), for l = 0..hy.  tw: W^l for l = 0..hy, then the
// stage twiddles of the hy-point FFT (the grid's stw_y table).  The first
// lanes of wave 0 transform; hy = 2^LOG2.
// The twiddles wait in LDS while the partials are summed (in the transforming
// lanes' registers they would halve the waves that do the summing).
// LDS of the row-forward workgroup: W^l, l = 0..hy, the stage twiddles [hy],
// the FFT buffer [hy] and rho [ny].
template <typename T>
__host__ __device__ constexpr size_t rows_fwd_lds(int ny, int my)
{
    return sizeof(cx<T>) * (size_t)(my + my / 2 + 1) + sizeof(T) * (size_t)ny;
}

template <typename T, bool FROM_PARTIALS, int NT, int LOG2>
__device__ __forceinline__ void rows_fwd_body(const DepositTarget &dep, int nblocks,
                                              const int64_t *__restrict__ q, double scale, int nx,
                                              int ny, const cx<T> *__restrict__ tw,
                                              cx<T> *__restrict__ at, int i, bool pipe,
                                              unsigned long long *red)
{
    using Fft = WaveFft<T, LOG2>;
    constexpr int half = Fft::L, my = 2 * half;  // hy: complex FFT length
    extern __shared__ __align__(16) unsigned char smem_raw[];
    cx<T> *twl = reinterpret_cast<cx<T> *>(smem_raw);  // W^l, l = 0..hy
    cx<T> *st = twl + half + 1;                        // hy
    cx<T> *z = st + half;                              // hy
    T *rho = reinterpret_cast<T *>(z + half);         // ny
    const int tid = threadIdx.x;
    // one round of loads: twiddles, and the carries or the dense row (ny <= NT)
    const int64_t qv = (!FROM_PARTIALS && tid < ny) ? q[(size_t)i * ny + tid] : 0;
    const unsigned long long cv =
        (FROM_PARTIALS && tid < ny) ? dep.carry[(size_t)i * ny + tid] : 0ull;
    for (int e = tid; e <= half + stage_twiddle_count(half, LOG2); e += NT) twl[e] = tw[e];
    if (FROM_PARTIALS) {
        const unsigned long long t = reduce_row<NT>(dep, red, nblocks, i, ny, tid, cv);
        if (tid < ny) rho[tid] = (T)((double)t * scale);
    } else {
        if (tid < ny) rho[tid] = (T)((double)qv * scale);
    }
    __syncthreads();
    // the row as a real sequence of length my: zero-padded (open boundary),
    // or odd-extended about the walls at j = 0 and j = ny (grounded pipe; the
    // wall row i = 0 and the wall column j = 0 take no charge)
    auto sample = [&](int l) -> T {
        if (!pipe) return l < ny ? rho[l] : T(0);
        if (i == 0 || l == 0 || l == ny) return T(0);
        return l < ny ? rho[l] : -rho[my - l];
    };
    if (tid < Fft::G) {
        cx<T> v[Fft::E];
#pragma unroll
        for (int r = 0; r < Fft::E; ++r) {
            const int m = tid + Fft::G * r;
            v[r] = cx<T>{sample(2 * m), sample(2 * m + 1)};
        }
        Fft fft;
        fft.load(st, tid);
        fft.run(v, z, tid);
#pragma unroll
        for (int r = 0; r < Fft::E; ++r) z[sw(tid + Fft::G * r)] = v[r];
    }
    __syncthreads();
    for (int l = tid; l <= half; l += NT) {
        const cx<T> zl = z[sw(l & (half - 1))];
        const cx<T> zm = conj(z[sw((half - l) & (half - 1))]);
        const cx<T> s = zl + zm, d = zl - zm;
        const cx<T> wd = mul_neg_i(twiddle(d, twl[l]));
        at[(size_t)l * nx + i] = scale_c(s + wd, T(0.5));
    }
}

// Line density of a long bunch (Sec. IV): sum the nblocks per-workgroup
// histograms of the last depositing pass exactly and write the node tables
//   lw[k] = h[k] / max h,   ld[k] = (h[k+1] - h[k-1]) / (2 dz max h)
// (h = 0 beyond the line; all zero for an empty line).  NT / nz groups of
// threads split the workgroups; acc is NT words of dynamic LDS.
template <int NT>
__device__ __forceinline__ void line_table_body(const LineSpec &L, int nblocks)
{
    extern __shared__ __align__(16) unsigned char smem_raw[];
    unsigned long long *acc = reinterpret_cast<unsigned long long *>(smem_raw);
    __shared__ unsigned long long wmax[NT / 64];
    const int tid = threadIdx.x, nz = L.nz;
    const int groups = NT / nz;
    const int k = tid % nz, g = tid / nz;
    unsigned long long s = 0;
    if (g < groups)
        for (int b0 = g; b0 < nblocks; b0 += 8 * groups) {
            unsigned long long v[8];  // eight loads in flight per round
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                const int b = b0 + u * groups;
                v[u] = b < nblocks ? L.partial[(size_t)b * nz + k] : 0ull;
            }
#pragma unroll
            for (int u = 0; u < 8; ++u) s += v[u];
        }
    acc[tid] = s;
    __syncthreads();
    unsigned long long h = 0;
    if (tid < nz)
        for (int r = 0; r < groups; ++r) h += acc[r * nz + tid];
    __syncthreads();
    if (tid < nz) acc[tid] = h;
    unsigned long long m = h;
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
        const unsigned long long v = __shfl_xor(m, o, 64);
        m = v > m ? v : m;
    }
    if ((tid & 63) == 0) wmax[tid >> 6] = m;
    __syncthreads();
    unsigned long long hmax = 0;
    for (int w = 0; w < NT / 64; ++w) hmax = wmax[w] > hmax ? wmax[w] : hmax;
    if (tid < nz) {
        double lw = 0.0, ld = 0.0;
        if (hmax) {
            const long long up = tid + 1 < nz ? (long long)acc[tid + 1] : 0;
            const long long down = tid > 0 ? (long long)acc[tid - 1] : 0;
            lw = (double)h / (double)hmax;
            ld = (double)(up - down) / (2.0 * L.dz * (double)hmax);
        }
        L.lw[tid] = lw;
        L.ld[tid] = ld;
    }
}

// Rows of the charge grid (LOG2: of the half length hy); with a line density
// (line.nz > 0) one more workgroup, index nx, reduces the line histograms.
template <typename T, bool FROM_PARTIALS, int LOG2>
__global__ void __launch_bounds__(kRowThreads, 8)
    k_rows_fwd(DepositTarget dep, int nblocks, const int64_t *__restrict__ q, double scale,
               int nx, int ny, const cx<T> *__restrict__ tw, cx<T> *__restrict__ at, bool pipe,
               LineSpec line)
{
    __shared__ unsigned long long red[FROM_PARTIALS ? kRowThreads * 4 : 1];
    if (line.nz > 0 && (int)blockIdx.x == nx) {
        line_table_body<kRowThreads>(line, nblocks);
        return;
    }
    rows_fwd_body<T, FROM_PARTIALS, kRowThreads, LOG2>(dep, nblocks, q, scale, nx, ny, tw, at,
                                                       (int)blockIdx.x, pipe, red);
}

// Every beam of a batch: workgroup -> (beam, row) from the batch's row table;
// the rows come from the partials of the beam's last batched pass.  A beam's
// row has few partial slices, so a smaller workgroup does it and more of them
// fit on a compute unit at once: NT threads, at least the largest ny and hy
// of the batch (128 when every beam's grid has ny <= 128, else 256).
template <typename T, int NT>
__global__ void __launch_bounds__(NT) k_rows_fwd_batched(BatchLaunch b)
{
    __shared__ unsigned long long red[NT * 4];
    const BatchInstance &I = b.inst[b.row_inst[blockIdx.x]];
    with_log2<3, NT == 128 ? 7 : 8>(I.log2_my - 1, [&](auto log2) {
        rows_fwd_body<T, true, NT, decltype(log2)::value>(
            I.dep, I.pass_blocks, nullptr, I.scale, I.nx, I.ny, (const cx<T> *)I.stw_y,
            (cx<T> *)I.spec_a, (int)blockIdx.x - I.row_block0, false, red);
    });
}

// What the column kernels read and write of one grid.
template <typename T>
struct ColumnArgs {
    const cx<T> *at;  // row spectra [hy+1][nx]
    const cx<T> *tw;  // stage twiddles of the mx-point FFT
    const T *ghat_t, *sx, *sy;
    cx<T> *b;         // (Bx, By) pairs [nx][hy+1]
    cx<T> *bp;        // the potential's column-inverse spectrum, or null
    int nx, hy;
    bool pipe;
};

// Column l (of hy + 1) of the row spectra in one group of G lanes: forward
// FFT along x, times the Green's spectrum, then one of the two differentiated
// inverse transforms (dir 0: x, dir 1: y); the two groups of a column both
// run the forward transform, which costs nothing while one of them would only
// wait, and then no group waits for another.  The forward transform's output
// is in the lanes that the inverse's first stage reads it in, so the product
// stays in registers.  dir 1 also gives the column-inverse of the potential's
// spectrum before the y difference to bp, when not null, for the node
// potential, on rows -1..nx (row i at bp[(i + 1) * (hy + 1)]; row -1 is the
// periodic row mx - 1, which the zero padding or the odd extension makes the
// potential's value one node outside the grid).
template <typename T, int LOG2>
__device__ __forceinline__ void column(const ColumnArgs<T> &c, int l, int dir, int t, cx<T> *buf)
{
    using Fft = WaveFft<T, LOG2>;
    constexpr int mx = Fft::L, E = Fft::E, G = Fft::G;
    const bool live = l <= c.hy;  // the last workgroup's spare groups store nothing
    if (!live) l = c.hy;
    const cx<T> *col = c.at + (size_t)l * c.nx;
    const T *g = c.ghat_t + (size_t)l * mx;
    // every input of the column in one round of loads
    cx<T> v[E];
    T vg[E], vs[E];
#pragma unroll
    for (int r = 0; r < E; ++r) {
        const int k = t + G * r;
        // zero-padded column (open boundary), or its odd extension about
        // the walls at i = 0 and i = nx (grounded pipe)
        const int src = column_source(k, c.nx, mx, c.pipe);
        const cx<T> z = src < 0 ? cx<T>{T(0), T(0)} : col[src];
        v[r] = (c.pipe && k > c.nx) ? cx<T>{-z.re, -z.im} : z;
    }
    Fft fft;
    fft.load(c.tw, t);
#pragma unroll
    for (int r = 0; r < E; ++r) {
        vg[r] = g[t + G * r];
        vs[r] = dir == 0 ? c.sx[t + G * r] : T(0);
    }
    const T syl = c.sy[l];
    fft.run(v, buf, t);
    // Inverse transforms as conj(FFT(conj(.))) of the conjugated inputs.
#pragma unroll
    for (int r = 0; r < E; ++r) {
        const cx<T> phi = scale_c(v[r], vg[r]);
        v[r] = dir == 0 ? conj(mul_neg_i(scale_c(phi, vs[r]))) : conj(phi);
    }
    fft.run(v, buf, t);
    if (!live) return;
#pragma unroll
    for (int r = 0; r < E; ++r) {
        const int i = t + G * r;
        const cx<T> u = conj(v[r]);
        if (i < c.nx)
            c.b[2 * ((size_t)i * (c.hy + 1) + l) + dir] =
                dir == 0 ? u : mul_neg_i(scale_c(u, syl));
        if (c.bp && dir == 1 && (i <= c.nx || i == mx - 1))
            c.bp[(size_t)(i <= c.nx ? i + 1 : 0) * (c.hy + 1) + l] = u;
    }
}

// Threads of a single-beam column workgroup: one wave when it holds a
// column's two groups, else two.
template <int LOG2>
constexpr int column_threads()
{
    return WaveFft<float, LOG2>::G > 32 ? 2 * WaveFft<float, LOG2>::G : 64;
}

template <typename T, int LOG2>
__global__ void __launch_bounds__(column_threads<LOG2>()) k_cols(ColumnArgs<T> c)
{
    using Fft = WaveFft<T, LOG2>;
    extern __shared__ __align__(16) unsigned char smem_raw[];
    const int group = threadIdx.x / Fft::G;
    constexpr int kColumns = column_threads<LOG2>() / (2 * Fft::G);
    column<T, LOG2>(c, (int)blockIdx.x * kColumns + (group >> 1), group & 1,
                    threadIdx.x % Fft::G,
                    reinterpret_cast<cx<T> *>(smem_raw) + (size_t)group * Fft::L);
}

// Every beam of a batch: kLineThreads / (2 G) neighbouring columns per
// workgroup; FFT lengths up to 2^MAXLOG.
template <typename T, int MAXLOG>
__global__ void __launch_bounds__(kLineThreads) k_cols_batched(BatchLaunch b)
{
    extern __shared__ __align__(16) unsigned char smem_raw[];
    const BatchInstance &I = b.inst[b.col_inst[blockIdx.x]];
    const ColumnArgs<T> c{(const cx<T> *)I.spec_a, (const cx<T> *)I.stw_x, (const T *)I.ghat_t,
                          (const T *)I.sx, (const T *)I.sy, (cx<T> *)I.spec_b, nullptr,
                          I.nx, I.my >> 1, false};
    with_log2<4, MAXLOG>(I.log2_mx, [&](auto log2) {
        using Fft = WaveFft<T, decltype(log2)::value>;
        const int group = threadIdx.x / Fft::G;
        constexpr int kColumns = kLineThreads / (2 * Fft::G);
        column<T, decltype(log2)::value>(
            c, ((int)blockIdx.x - I.col_block0) * kColumns + (group >> 1), group & 1,
            threadIdx.x % Fft::G, reinterpret_cast<cx<T> *>(smem_raw) + (size_t)group * Fft::L);
    });
}

// Row i in one group of G lanes: Z[l] = Bx[l] + i By[l] for l = 0..hy and
// Z[my-l] = conj(Bx[l]) + i conj(By[l]) for 0 < l < hy (hy = my / 2); one
// inverse FFT gives ex + i ey on the first ny entries (tw: the stage twiddles
// of the my-point FFT).  Written either as two arrays (ex, ey) or interleaved
// into ef (Ex, Ey per node).
template <typename T, int LOG2>
__device__ __forceinline__ void field_row(const cx<T> *__restrict__ b, int nx, int ny,
                                          const cx<T> *__restrict__ tw, T *__restrict__ ex,
                                          T *__restrict__ ey, cx<T> *__restrict__ ef, int i, int t,
                                          cx<T> *buf)
{
    using Fft = WaveFft<T, LOG2>;
    constexpr int my = Fft::L, hy = my / 2;
    const bool live = i >= 0 && i < nx;  // spare groups read row 0, store nothing
    const cx<T> *row = b + 2 * (size_t)(live ? i : 0) * (hy + 1);
    cx<T> v[Fft::E];
#pragma unroll
    for (int r = 0; r < Fft::E; ++r) {
        const int e = t + Fft::G * r, l = e <= hy ? e : my - e;
        const cx<T> X = row[2 * l], Y = row[2 * l + 1];
        // conjugated inputs for conj(FFT(conj(.)))
        v[r] = e <= hy ? conj(X + mul_pos_i(Y)) : conj(conj(X) + mul_pos_i(conj(Y)));
    }
    Fft fft;
    fft.load(tw, t);
    fft.run(v, buf, t);
#pragma unroll
    for (int r = 0; r < Fft::E; ++r) {
        const int j = t + Fft::G * r;
        if (!live || j >= ny) continue;
        const cx<T> z = conj(v[r]);
        if (ef) {
            ef[(size_t)i * ny + j] = z;
        } else {
            ex[(size_t)i * ny + j] = z.re;
            ey[(size_t)i * ny + j] = z.im;
        }
    }
}

// Row i (-1..nx) of the node potential on columns -1..ny
// (phi[(i + 1) * (ny + 2) + j + 1]) from the potential's column-inverse
// spectrum: one inverse FFT of its Hermitian row.
template <typename T, int LOG2>
__device__ __forceinline__ void potential_row(const cx<T> *__restrict__ bp, int ny,
                                              const cx<T> *__restrict__ tw, T *__restrict__ phi,
                                              int i, int t, cx<T> *buf)
{
    using Fft = WaveFft<T, LOG2>;
    constexpr int my = Fft::L, hy = my / 2;
    const cx<T> *row = bp + (size_t)(i + 1) * (hy + 1);
    cx<T> v[Fft::E];
#pragma unroll
    for (int r = 0; r < Fft::E; ++r) {
        const int e = t + Fft::G * r;
        v[r] = e <= hy ? conj(row[e]) : row[my - e];
    }
    Fft fft;
    fft.load(tw, t);
    fft.run(v, buf, t);
    T *out = phi + (size_t)(i + 1) * (ny + 2);
#pragma unroll
    for (int r = 0; r < Fft::E; ++r) {
        const int j = t + Fft::G * r;
        if (j <= ny || j == my - 1) out[j <= ny ? j + 1 : 0] = v[r].re;
    }
}

// One wave of field rows per workgroup; with the potential (bp) the last
// nx + 2 groups of rows are the potential's rows -1..nx.
template <typename T, int LOG2>
__global__ void __launch_bounds__(64)
    k_rows_inv(const cx<T> *__restrict__ b, int nx, int ny, const cx<T> *__restrict__ tw,
               T *__restrict__ ex, T *__restrict__ ey, cx<T> *__restrict__ ef,
               const cx<T> *__restrict__ bp, T *__restrict__ phi)
{
    using Fft = WaveFft<T, LOG2>;
    extern __shared__ __align__(16) unsigned char smem_raw[];
    constexpr int kRows = 64 / Fft::G;
    const int group = threadIdx.x / Fft::G, t = threadIdx.x % Fft::G;
    cx<T> *buf = reinterpret_cast<cx<T> *>(smem_raw) + (size_t)group * Fft::L;
    const int field_blocks = (nx + kRows - 1) / kRows, blk = (int)blockIdx.x;
    if (blk < field_blocks) {
        field_row<T, LOG2>(b, nx, ny, tw, ex, ey, ef, blk * kRows + group, t, buf);
    } else {
        // spare groups of the last workgroup repeat row nx
        const int i = (blk - field_blocks) * kRows + group - 1;
        potential_row<T, LOG2>(bp, ny, tw, phi, i < nx ? i : nx, t, buf);
    }
}

// Every beam of a batch: kLineThreads / G rows per workgroup; FFT lengths up
// to 2^MAXLOG.
template <typename T, int MAXLOG>
__global__ void __launch_bounds__(kLineThreads) k_rows_inv_batched(BatchLaunch b)
{
    extern __shared__ __align__(16) unsigned char smem_raw[];
    const BatchInstance &I = b.inst[b.inv_inst[blockIdx.x]];
    with_log2<4, MAXLOG>(I.log2_my, [&](auto log2) {
        using Fft = WaveFft<T, decltype(log2)::value>;
        const int group = threadIdx.x / Fft::G;
        constexpr int kRows = kLineThreads / Fft::G;
        field_row<T, decltype(log2)::value>(
            (const cx<T> *)I.spec_b, I.nx, I.ny, (const cx<T> *)I.stw_y + I.my + 1, nullptr,
            nullptr, (cx<T> *)I.ef, ((int)blockIdx.x - I.inv_block0) * kRows + group,
            threadIdx.x % Fft::G, reinterpret_cast<cx<T> *>(smem_raw) + (size_t)group * Fft::L);
    });
}

template <typename T>
hipError_t launch_tail(hipStream_t s, const SolveWorkspace &w, void *ex, void *ey, void *ef)
{
    const bool want_phi = w.want_phi;
    const ColumnArgs<T> c{(const cx<T> *)w.spec_a, (const cx<T> *)w.stw_x, (const T *)w.ghat_t,
                          (const T *)w.sx, (const T *)w.sy, (cx<T> *)w.spec_b,
                          want_phi ? (cx<T> *)w.spec_p : nullptr, w.nx, w.my / 2, w.pipe};
    with_log2<4, 9>(w.log2_mx, [&](auto log2) {
        constexpr int LOG2 = decltype(log2)::value, NT = column_threads<LOG2>();
        using Fft = WaveFft<T, LOG2>;
        constexpr int kColumns = NT / (2 * Fft::G);
        hipLaunchKernelGGL((k_cols<T, LOG2>), dim3((c.hy + kColumns) / kColumns), dim3(NT),
                           sizeof(cx<T>) * NT * Fft::E, s, c);
    });
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    with_log2<4, 9>(w.log2_my, [&](auto log2) {
        constexpr int LOG2 = decltype(log2)::value;
        using Fft = WaveFft<T, LOG2>;
        constexpr int kRows = 64 / Fft::G;
        const int blocks = (w.nx + kRows - 1) / kRows + (want_phi ? (w.nx + 1 + kRows) / kRows : 0);
        hipLaunchKernelGGL((k_rows_inv<T, LOG2>), dim3(blocks), dim3(64),
                           sizeof(cx<T>) * 64 * Fft::E, s, (const cx<T> *)w.spec_b,
                           w.nx, w.ny, (const cx<T> *)w.stw_y + w.my + 1, (T *)ex, (T *)ey,
                           (cx<T> *)ef, (const cx<T> *)c.bp, want_phi ? (T *)w.phi : (T *)nullptr);
    });
    return hipGetLastError();
}

template <typename T, bool FROM_PARTIALS>
hipError_t launch_solve_t(hipStream_t s, const SolveWorkspace &w, const DepositTarget &dep,
                          int nblocks, const int64_t *q, double scale, void *ex, void *ey,
                          void *ef)
{
    // the line tables come from the partials of a depositing pass only
    LineSpec line = FROM_PARTIALS ? w.line : LineSpec{};
    size_t row_lds = rows_fwd_lds<T>(w.ny, w.my);
    if (line.nz > 0) row_lds = std::max(row_lds, sizeof(unsigned long long) * (size_t)kRowThreads);
    with_log2<3, 8>(w.log2_my - 1, [&](auto log2) {
        hipLaunchKernelGGL((k_rows_fwd<T, FROM_PARTIALS, decltype(log2)::value>),
                           dim3(w.nx + (line.nz > 0 ? 1 : 0)), dim3(kRowThreads), row_lds, s, dep,
                           nblocks, q, scale, w.nx, w.ny, (const cx<T> *)w.stw_y,
                           (cx<T> *)w.spec_a, w.pipe, line);
    });
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    return launch_tail<T>(s, w, ex, ey, ef);
}

// LDS of a batched column or row-inverse workgroup: kLineThreads lanes of 4
// elements each (8 when a beam's FFT has 512 points).  The kernels for batches
// without such a beam leave the 512-point code, and its registers, out.
template <typename T>
hipError_t launch_solve_batched_t(hipStream_t s, const BatchLaunch &b, const BatchGridShape &g)
{
    const size_t row_lds = rows_fwd_lds<T>(g.max_ny, g.max_my);
    constexpr size_t line_lds = sizeof(cx<T>) * kLineThreads * 4;
    if (g.max_ny <= 128 && g.max_my / 2 <= 128)
        hipLaunchKernelGGL((k_rows_fwd_batched<T, 128>), dim3(g.rows), dim3(128), row_lds, s, b);
    else
        hipLaunchKernelGGL((k_rows_fwd_batched<T, 256>), dim3(g.rows), dim3(256), row_lds, s, b);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    if (g.max_mx <= 256)
        hipLaunchKernelGGL((k_cols_batched<T, 8>), dim3(g.col_blocks), dim3(kLineThreads),
                           line_lds, s, b);
    else
        hipLaunchKernelGGL((k_cols_batched<T, 9>), dim3(g.col_blocks), dim3(kLineThreads),
                           2 * line_lds, s, b);
    e = hipGetLastError();
    if (e != hipSuccess) return e;
    if (g.max_my <= 256)
        hipLaunchKernelGGL((k_rows_inv_batched<T, 8>), dim3(g.inv_blocks), dim3(kLineThreads),
                           line_lds, s, b);
    else
        hipLaunchKernelGGL((k_rows_inv_batched<T, 9>), dim3(g.inv_blocks), dim3(kLineThreads),
                           2 * line_lds, s, b);
    return hipGetLastError();
}

}  // namespace

// Lanes of an FFT of length 2^log2 (any precision).
static int fft_lanes(int log2) { return (1 << log2) / (log2 == 9 ? 8 : 4); }

int batch_column_blocks(int log2_mx, int hy)
{
    const int columns = kLineThreads / (2 * fft_lanes(log2_mx));
    return (hy + columns) / columns;
}

int batch_inverse_blocks(int log2_my, int nx)
{
    const int rows = kLineThreads / fft_lanes(log2_my);
    return (nx + rows - 1) / rows;
}

hipError_t launch_solve_batched(hipStream_t s, const BatchLaunch &b, bool mixed,
                                const BatchGridShape &g)
{
    return mixed ? launch_solve_batched_t<float>(s, b, g) : launch_solve_batched_t<double>(s, b, g);
}

hipError_t launch_reduce(hipStream_t s, const DepositTarget &dep, int blocks_used, int nx, int ny,
                         int64_t *q, int64_t *n_in)
{
    hipLaunchKernelGGL(k_reduce, dim3(nx), dim3(kRowThreads), 0, s, dep, blocks_used, nx, ny, q,
                       n_in);
    return hipGetLastError();
}

hipError_t launch_solve(hipStream_t s, const SolveWorkspace &w, const int64_t *q, double scale,
                        void *ex, void *ey, void *ef)
{
    DepositTarget none{};
    return w.mixed ? launch_solve_t<float, false>(s, w, none, 0, q, scale, ex, ey, ef)
                   : launch_solve_t<double, false>(s, w, none, 0, q, scale, ex, ey, ef);
}

hipError_t launch_solve_partials(hipStream_t s, const SolveWorkspace &w, const DepositTarget &dep,
                                 int blocks_used, double scale, void *ef)
{
    return w.mixed ? launch_solve_t<float, true>(s, w, dep, blocks_used, nullptr, scale, nullptr,
                                                 nullptr, ef)
                   : launch_solve_t<double, true>(s, w, dep, blocks_used, nullptr, scale, nullptr,
                                                  nullptr, ef);
}

}  // namespace scpic
