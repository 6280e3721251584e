// Column-slab hierarchy of a CSR matrix: the analysis step that builds it and the first step of the
// SpMV over it.
//
// Why: on this chip a 4-byte gather of x that misses the 32 KB L1 costs one 64-byte request slot of the
// L1's miss path whatever the table's size, and a row-ordered CSR with scattered columns misses almost
// always.  Section 8.6 of the paper gets locality by tiling (split a loop, move the outer part outward);
// Section 3 lets the position cut be taken in any coordinate hierarchy.  Here the column loop j is split
// by a slab of PSK_SLAB_COLS columns, jo = j / PSK_SLAB_COLS moves outermost and A is STORED in that
// order once (three levels: jo dense, i compressed, ji compressed).  The position space of the leaf
// level is then cut into equal pieces as before, but a piece now needs only one slab of x, which a
// workgroup keeps in on-chip memory (128 KB of the CU's 160 KB): gathers become LDS reads.
//
// Structure (all built here, on the device; the CPU oracle builds the same arrays from the definition):
//   slots   = the stored entries sorted by (slab, CSR position): a stable bucketing; every slab is
//             padded to a multiple of PSK_SLAB_CHUNK slots so that a chunk never crosses a slab;
//   pair    = a maximal run of slots of one row inside one chunk; scol bit 15 marks a pair's last slot;
//   step 1  : P[pair] = sum of value * x over the pair's slots            (k_slab_pairs, this file)
//   step 2  : y[i] = sum of P over the pairs of row i, listed by (qpos, qidx): the ordinary position-cut
//             SpMV kernel with unit values (k_spmv_pos, VARIANT 6).
// A chunk is one wave's unit of work: no sum crosses a chunk, so step 1 needs no communication between
// waves, no carries and no barrier except when a workgroup moves on to the next slab.
#include "psk_dev.h"
#include "psk_internal.h"

namespace psk {

constexpr int SLAB_CH = kSlabChunk;
constexpr int BUILD_BT = kSlabBuildBlock;     // CSR positions per block of the bucketing kernels

// Per value type: columns per slab (what fits into the LDS next to the staging area) and values per 16 bytes.
typedef double v2d __attribute__((ext_vector_type(2)));
template <typename T> struct SlabOf;
template <> struct SlabOf<float>  { static constexpr int W = kSlabCols,    G = 4, WAVES = 16, STAGE = SLAB_CH; typedef v4f V; };
template <> struct SlabOf<double> { static constexpr int W = kSlabColsF64, G = 2, WAVES = 16, STAGE = SLAB_CH / 2; typedef v2d V; };

// Where the value of slot j is stored.  A lane of the pair kernel owns 8 consecutive slots of a chunk; stored in
// slot order its 16-byte loads would each touch every other 16 bytes of the chunk.  Inside each chunk the values
// are therefore stored in groups of G = 16 bytes / value size: [first G slots of lane 0, of lane 1, ... | next G
// slots of lane 0, ...], so that every load is contiguous over the wave (measured for fp32 on the streams alone: 60
// instead of 65 us).
template <int G>
__host__ __device__ __forceinline__ int slab_value_index(int j)
{
    const int o = j & (SLAB_CH - 1), l = o >> 3, k = o & 7;
    return (j - o) + (k / G) * (SLAB_CH / 8 * G) + G * l + (k % G);
}

// ------------------------------------------------------------------ DPP scans over the 64 lanes of a wave
template <int CTRL, int ROWMASK>
__device__ __forceinline__ int dpp_i(int v) { return __builtin_amdgcn_update_dpp(0, v, CTRL, ROWMASK, 0xF, false); }
template <int CTRL, int ROWMASK>
__device__ __forceinline__ float dpp_f(float v)
{
    return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), CTRL, ROWMASK, 0xF, false));
}
template <int CTRL, int ROWMASK>
__device__ __forceinline__ double dpp_f(double v)
{
    const long long b = __builtin_bit_cast(long long, v);
    const unsigned lo = (unsigned)dpp_i<CTRL, ROWMASK>((int)(unsigned)b), hi = (unsigned)dpp_i<CTRL, ROWMASK>((int)(b >> 32));
    return __builtin_bit_cast(double, (long long)(((unsigned long long)hi << 32) | lo));
}
// row_shr 1, 2, 4, 8 scan each row of 16 lanes; row_bcast15 hands lane 15 of rows 0 and 2 to rows 1 and 3,
// row_bcast31 hands lane 31 to rows 2 and 3.  Lanes without a source receive 0.
__device__ __forceinline__ int wave_scan_add(int v)
{
    v += dpp_i<0x111, 0xF>(v);
    v += dpp_i<0x112, 0xF>(v);
    v += dpp_i<0x114, 0xF>(v);
    v += dpp_i<0x118, 0xF>(v);
    v += dpp_i<0x142, 0xA>(v);
    v += dpp_i<0x143, 0xC>(v);
    return v;
}
// bits of `mask` that belong to lanes below this one
__device__ __forceinline__ int lanes_below(unsigned long long mask)
{
    return (int)__builtin_amdgcn_mbcnt_hi((unsigned)(mask >> 32), __builtin_amdgcn_mbcnt_lo((unsigned)mask, 0u));
}
// Inclusive segmented sum: a lane with f != 0 starts afresh (takes nothing from the lanes below it).
template <typename T>
__device__ __forceinline__ T wave_segscan(T v, int f)
{
#define PSK_SEG_STEP(CTRL, MASK)                       \
    {                                                  \
        const T pv = dpp_f<CTRL, MASK>(v);             \
        const int pf = dpp_i<CTRL, MASK>(f);           \
        v = f ? v : v + pv;                            \
        f |= pf;                                       \
    }
    PSK_SEG_STEP(0x111, 0xF) PSK_SEG_STEP(0x112, 0xF) PSK_SEG_STEP(0x114, 0xF) PSK_SEG_STEP(0x118, 0xF)
    PSK_SEG_STEP(0x142, 0xA) PSK_SEG_STEP(0x143, 0xC)
#undef PSK_SEG_STEP
    return v;
}

// ------------------------------------------------------------------ step 1 of the product
// Persistent workgroups: every workgroup owns one piece of cpw consecutive chunks (the position space DIVIDED into
// equal pieces, Section 5), walks them slab by slab, loads the slab's part of x into LDS once and lets its
// 16 waves take the chunks of that slab round-robin.  A lane owns 8 consecutive slots (two 16-byte loads of
// values, one of columns); the next chunk's loads are issued before the current one is processed.
// Inside a chunk (no branches): the lane walks its 8 slots with a running sum that restarts after a pair
// end and writes every running sum to LDS -- to the pair's place in the chunk (number of pair ends before
// it) when the slot ends a pair, to a dummy word otherwise; a segmented DPP scan then hands each lane the
// open sum of the lanes below it, which is added to the lane's first pair.  The chunk's pair sums, now
// compact in LDS, leave with full-width coalesced stores to P[chunk_pair[c] ...].
// LDS: 127.9 KB of x + 2 KB of pair sums per wave + the dummy words = the CU's 160 KB.  fp64: 127.75 KB of x = 16 352 columns and
// room for the sums of half a chunk's slots, which leave in two rounds where a chunk has more pairs (with few entries per pair),
// so that 16 waves fit: eight waves of a whole chunk each left the vector units waiting.  Power-law configuration 186.1 -> 178.4 us per
// product; 400 000 rows x 3 M columns, power-law 47.7 -> 42.7; uniform, 10 per row x 3 M (two rounds in most chunks) 90.2 -> 86.8.
template <typename T>
__global__ __launch_bounds__(SlabOf<T>::WAVES * WAVE) void k_slab_pairs(const T *__restrict__ svals,
                                                     const unsigned short *__restrict__ scol,
                                                     const int *__restrict__ chunk_pair,
                                                     const int *__restrict__ slab_chunk,
                                                     const T *__restrict__ x, T *__restrict__ P, int cols,
                                                     int nslabs, int nchunks, int cpw)
{
    constexpr int WAVES = SlabOf<T>::WAVES;
    constexpr int STAGE = SlabOf<T>::STAGE;
    constexpr int W = SlabOf<T>::W, G = SlabOf<T>::G, NV = 8 / G;      // NV 16-byte loads of values per lane
    typedef typename SlabOf<T>::V V;
    __shared__ T xs[W];
    __shared__ T stage[WAVES * STAGE + 32];           // + one dummy word per LDS bank
    static_assert(sizeof(T) * (W + WAVES * STAGE + 32) <= 163840, "the window and the staging area fill the CU's LDS");
    const int tid = threadIdx.x, lane = tid & (WAVE - 1);
    const int wave = __builtin_amdgcn_readfirstlane(tid / WAVE);
    T *st = stage + wave * STAGE;
    const int dummy = (WAVES - wave) * STAGE + (lane & 31);      // index, relative to st, of a word nobody reads
    // piece of this workgroup: neighbouring pieces go to workgroups of the same die, so that the slabs of x they share
    // are fetched into that die's L2 once (measured on the power-law matrix: 76.2 against 79.4 us)
    const int piece = xcd_tile(blockIdx.x, (nchunks + cpw - 1) / cpw);
    if (piece < 0) return;
    int c0 = piece * cpw;
    const int c1 = min(c0 + cpw, nchunks);
    if (c0 >= c1) return;
    PSK_TRACE_WORKGROUP();
    int s;      // slab of chunk c0: max { s : slab_chunk[s] <= c0 }
    {
        int lo = 0, hi = nslabs;
        while (lo < hi) {
            const int mid = lo + ((hi - lo + 1) >> 1);
            if (slab_chunk[mid] <= c0) lo = mid; else hi = mid - 1;
        }
        s = lo;
    }
    while (c0 < c1) {
        while (slab_chunk[s + 1] <= c0) ++s;            // skips empty slabs; c0 < nchunks = slab_chunk[nslabs]
        const int ce = min(c1, slab_chunk[s + 1]);
        __syncthreads();                                  // the previous slab's window is no longer read
        const long long xb = (long long)s * W;
        const int wlen = (int)min((long long)W, (long long)cols - xb);
        const bool x16 = (reinterpret_cast<uintptr_t>(x + xb) & 15) == 0;
        for (int i = tid * G; i < wlen; i += WAVES * WAVE * G) {
            if (x16 && i + G <= wlen) {
                *reinterpret_cast<V *>(&xs[i]) = *reinterpret_cast<const V *>(x + xb + i);
            } else {
                for (int j = i; j < i + G && j < wlen; ++j) xs[j] = x[xb + j];
            }
        }
        __syncthreads();
        int c = c0 + wave;
        V va[NV];
#pragma unroll
        for (int g = 0; g < NV; ++g) va[g] = V{};
        v4i cc = {0, 0, 0, 0};
        int pb = 0;
        auto issue = [&](int ci) {
            const long long b = (long long)ci * SLAB_CH;
#pragma unroll
            for (int g = 0; g < NV; ++g)                                       // slots 8*lane + g*G .. + G-1
                va[g] = ld_stream(reinterpret_cast<const V *>(svals + b + g * (SLAB_CH / 8 * G) + lane * G));
            cc = ld_stream(reinterpret_cast<const v4i *>(scol + b + lane * 8));
            // lanes 0 and 1 fetch the chunk's first pair and the next chunk's: a vector load on purpose, a scalar
            // load would share its counter with the LDS reads and make each of them wait for its round trip
            pb = chunk_pair[ci + (lane & 1)];
        };
        if (c < ce) issue(c);
        for (; c < ce; c += WAVES) {
            T v[8];
#pragma unroll
            for (int j = 0; j < 8; ++j) v[j] = va[j / G][j % G];
            const v4i q = cc;
            const int pbase = rl(pb, 0), np = rl(pb, 1) - pbase;
            if (c + WAVES < ce) issue(c + WAVES);
            const unsigned w0 = (unsigned)q.x, w1 = (unsigned)q.y, w2 = (unsigned)q.z, w3 = (unsigned)q.w;
            // bit j = slot j of this lane ends a pair (bit 15 of its 16-bit column word)
            const unsigned ends = ((w0 >> 15) & 1u) | ((w0 >> 30) & 2u) | ((w1 >> 13) & 4u) | ((w1 >> 28) & 8u) |
                                  ((w2 >> 11) & 16u) | ((w2 >> 26) & 32u) | ((w3 >> 9) & 64u) | ((w3 >> 24) & 128u);
            const unsigned w[4] = {w0, w1, w2, w3};
            T p[8];
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                const unsigned h = (j & 1) ? (w[j >> 1] >> 16) : w[j >> 1];
                p[j] = v[j] * xs[h & 0x7fffu];
            }
            const int cnt = __popc(ends);
            const int first = wave_scan_add(cnt) - cnt;         // place of this lane's first pair end in the chunk
            T run = 0, sum[8];
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                run += p[j];
                sum[j] = run;
                run = (ends >> j) & 1u ? T(0) : run;
            }
            // `run` is the lane's open sum; the lane below hands over the open sum of all lanes below it
            const T open = wave_segscan<T>(run, cnt ? 1 : 0);
            const T carry = __shfl_up(open, 1, WAVE);
            for (int k0 = 0; k0 < np; k0 += STAGE) {            // (one round unless the staging area is smaller than a chunk)
                int place = first - k0;
#pragma unroll
                for (int j = 0; j < 8; ++j) {
                    const bool e = (ends >> j) & 1u;
                    st[e && (STAGE == SLAB_CH || (unsigned)place < (unsigned)STAGE) ? place : dummy] = sum[j];
                    place += e ? 1 : 0;
                }
                // head + carry (a chunk's first slot starts a pair)
                if (cnt && lane && (STAGE == SLAB_CH || (unsigned)(first - k0) < (unsigned)STAGE)) st[first - k0] += carry;
                const int n = STAGE == SLAB_CH ? np : min(np - k0, STAGE);
                for (int k = lane; k < n; k += WAVE) P[pbase + k0 + k] = st[k];
            }
        }
        c0 = ce;
        ++s;
    }
}

template <typename T>
static hipError_t launch_slab_pairs_t(const T *svals, const uint16_t *scol, const int32_t *chunk_pair,
                                      const int32_t *slab_chunk, const T *x, T *P, int32_t cols, int32_t nslabs,
                                      int32_t nchunks, int32_t nwg, hipStream_t s)
{
    if (nchunks <= 0) return hipSuccess;
    if (nwg < 1) nwg = 1;
    const int cpw = (nchunks + nwg - 1) / nwg;
    const int grid = xcd_grid((nchunks + cpw - 1) / cpw);
    PSK_LAUNCH(k_slab_pairs<T>, dim3(grid), dim3(SlabOf<T>::WAVES * WAVE), 0, s, svals, scol, chunk_pair, slab_chunk, x, P, cols, nslabs,
               nchunks, cpw);
    return take_launch_status();
}

hipError_t launch_slab_pairs(const float *svals, const uint16_t *scol, const int32_t *chunk_pair,
                             const int32_t *slab_chunk, const float *x, float *P, int32_t cols, int32_t nslabs,
                             int32_t nchunks, int32_t nwg, hipStream_t s)
{
    return launch_slab_pairs_t<float>(svals, scol, chunk_pair, slab_chunk, x, P, cols, nslabs, nchunks, nwg, s);
}

hipError_t launch_slab_pairs_f64(const double *svals, const uint16_t *scol, const int32_t *chunk_pair,
                                 const int32_t *slab_chunk, const double *x, double *P, int32_t cols, int32_t nslabs,
                                 int32_t nchunks, int32_t nwg, hipStream_t s)
{
    return launch_slab_pairs_t<double>(svals, scol, chunk_pair, slab_chunk, x, P, cols, nslabs, nchunks, nwg, s);
}

// ------------------------------------------------------------------ prefix sums over int32 arrays
// Exclusive scans.  Three kernels: sums of blocks of 4096, a single-workgroup scan of those sums, then every block
// scans its own elements on top of its offset.  In place (out == in) is allowed.
constexpr int SCAN_EPT = 16, SCAN_BLOCK = 256 * SCAN_EPT;

__device__ __forceinline__ int block_scan_256(int v, int *s_w, int *total)
{
    // inclusive scan of one value per thread over 256 threads; s_w has 4 ints
    const int lane = threadIdx.x & (WAVE - 1), wave = threadIdx.x / WAVE;
    const int inc = wave_scan_add(v);
    if (lane == WAVE - 1) s_w[wave] = inc;
    __syncthreads();
    int off = 0;
    for (int w = 0; w < wave; ++w) off += s_w[w];
    *total = s_w[0] + s_w[1] + s_w[2] + s_w[3];
    __syncthreads();
    return inc + off;
}

// a thread's SCAN_EPT consecutive elements, as four 16-byte loads when they all exist (the arrays start on 256-byte
// boundaries and a thread's share on a 64-byte one)
template <bool NONZERO>
__device__ __forceinline__ void scan_load(const int *__restrict__ in, long long base, long long n, int (&v)[SCAN_EPT])
{
    if (base + SCAN_EPT <= n) {
#pragma unroll
        for (int g = 0; g < SCAN_EPT / 4; ++g) {
            const v4i t = *reinterpret_cast<const v4i *>(in + base + 4 * g);
            v[4 * g] = t.x; v[4 * g + 1] = t.y; v[4 * g + 2] = t.z; v[4 * g + 3] = t.w;
        }
    } else {
#pragma unroll
        for (int i = 0; i < SCAN_EPT; ++i) v[i] = base + i < n ? in[base + i] : 0;
    }
    if (NONZERO) {
#pragma unroll
        for (int i = 0; i < SCAN_EPT; ++i) v[i] = v[i] != 0;
    }
}

// NONZERO: the scanned sequence is (in[i] != 0)
template <bool NONZERO>
__global__ __launch_bounds__(256) void k_scan_reduce(const int *__restrict__ in, long long n, int *__restrict__ bsum)
{
    __shared__ int s_w[4];
    const long long base = (long long)blockIdx.x * SCAN_BLOCK + threadIdx.x * SCAN_EPT;
    int v[SCAN_EPT];
    scan_load<NONZERO>(in, base, n, v);
    int t = 0;
#pragma unroll
    for (int i = 0; i < SCAN_EPT; ++i) t += v[i];
    int total;
    block_scan_256(t, s_w, &total);
    if (threadIdx.x == 0) bsum[blockIdx.x] = total;
}

// exclusive scan of bsum[0 .. nb) in place, by one workgroup of 256 threads
__global__ __launch_bounds__(256) void k_scan_spine(int *__restrict__ bsum, long long nb)
{
    __shared__ int s_w[4];
    int carry = 0;
    for (long long b0 = 0; b0 < nb; b0 += 256) {
        const long long i = b0 + threadIdx.x;
        const int v = i < nb ? bsum[i] : 0;
        int total;
        const int inc = block_scan_256(v, s_w, &total);
        if (i < nb) bsum[i] = carry + inc - v;
        carry += total;
    }
}

template <bool NONZERO>
__global__ __launch_bounds__(256) void k_scan_apply(const int *__restrict__ in, int *__restrict__ out, long long n,
                                                    const int *__restrict__ bsum)
{
    __shared__ int s_w[4];
    const long long base = (long long)blockIdx.x * SCAN_BLOCK + threadIdx.x * SCAN_EPT;
    int v[SCAN_EPT];
    scan_load<NONZERO>(in, base, n, v);
    int t = 0;
#pragma unroll
    for (int i = 0; i < SCAN_EPT; ++i) t += v[i];
    int total;
    const int inc = block_scan_256(t, s_w, &total);
    int run = bsum[blockIdx.x] + inc - t;
    int o[SCAN_EPT];
#pragma unroll
    for (int i = 0; i < SCAN_EPT; ++i) {
        o[i] = run;
        run += v[i];
    }
    if (base + SCAN_EPT <= n) {
#pragma unroll
        for (int g = 0; g < SCAN_EPT / 4; ++g)
            *reinterpret_cast<v4i *>(out + base + 4 * g) = v4i{o[4 * g], o[4 * g + 1], o[4 * g + 2], o[4 * g + 3]};
    } else {
#pragma unroll
        for (int i = 0; i < SCAN_EPT; ++i)
            if (base + i < n) out[base + i] = o[i];
    }
}

size_t scan_tmp_ints(int64_t n) { return (size_t)((n + SCAN_BLOCK - 1) / SCAN_BLOCK) + 1; }

// exclusive scan of in[0 .. n) into out (in place allowed); nonzero: of the sequence (in[i] != 0)
static void launch_scan(const int32_t *in, int32_t *out, int64_t n, int32_t *bsum, bool nonzero, hipStream_t s)
{
    if (n <= 0) return;
    const long long nb = (n + SCAN_BLOCK - 1) / SCAN_BLOCK;
    if (nonzero) PSK_LAUNCH(k_scan_reduce<true>, dim3((unsigned)nb), dim3(256), 0, s, in, (long long)n, bsum);
    else PSK_LAUNCH(k_scan_reduce<false>, dim3((unsigned)nb), dim3(256), 0, s, in, (long long)n, bsum);
    PSK_LAUNCH(k_scan_spine, dim3(1), dim3(256), 0, s, bsum, nb);
    if (nonzero) PSK_LAUNCH(k_scan_apply<true>, dim3((unsigned)nb), dim3(256), 0, s, in, out, (long long)n, bsum);
    else PSK_LAUNCH(k_scan_apply<false>, dim3((unsigned)nb), dim3(256), 0, s, in, out, (long long)n, bsum);
}

// ------------------------------------------------------------------ the analysis step: CSR -> slab hierarchy
// H[s * nblk + b] = number of positions of block b (BUILD_BT consecutive CSR positions) that fall into slab s.
__global__ __launch_bounds__(256) void k_slab_hist(int nnz, const int *__restrict__ crd, int W, int nslabs, int nblk,
                                                   int *__restrict__ H)
{
    extern __shared__ int hist[];
    for (int s = threadIdx.x; s < nslabs; s += 256) hist[s] = 0;
    __syncthreads();
    const int b = blockIdx.x;
    const long long p0 = (long long)b * BUILD_BT;
    for (int i = threadIdx.x; i < BUILD_BT; i += 256)
        if (p0 + i < nnz) atomicAdd(&hist[crd[p0 + i] / W], 1);
    __syncthreads();
    for (int s = threadIdx.x; s < nslabs; s += 256) H[(long long)s * nblk + b] = hist[s];
}

// E = exclusive scan of H (E[nslabs * nblk] = nnz).  One workgroup: slab s holds E[(s+1)*nblk] - E[s*nblk]
// positions, padded to a multiple of the chunk; slab_chunk = exclusive scan of the padded sizes in chunks.
// meta[0] = number of slots.
__global__ __launch_bounds__(256) void k_slab_bases(const int *__restrict__ E, int nslabs, int nblk,
                                                    int *__restrict__ slab_chunk, int *__restrict__ meta)
{
    __shared__ int s_w[4];
    int carry = 0;
    for (int s0 = 0; s0 < nslabs; s0 += 256) {
        const int s = s0 + threadIdx.x;
        int chunks = 0;
        if (s < nslabs) {
            const int cnt = E[(long long)(s + 1) * nblk] - E[(long long)s * nblk];
            chunks = (cnt + SLAB_CH - 1) / SLAB_CH;
        }
        int total;
        const int inc = block_scan_256(chunks, s_w, &total);
        if (s < nslabs) slab_chunk[s] = carry + inc - chunks;
        carry += total;
    }
    if (threadIdx.x == 0) {
        slab_chunk[nslabs] = carry;
        meta[0] = carry * SLAB_CH;
    }
}

// The pad slots of slab s (fewer than a chunk): value 0, column 0, no row, no source position.
template <typename T>
__global__ __launch_bounds__(64) void k_slab_pads(const int *__restrict__ E, int nblk, const int *__restrict__ slab_chunk,
                                                  T *__restrict__ svals, unsigned short *__restrict__ scol,
                                                  int *__restrict__ srow, int *__restrict__ src)
{
    const int s = blockIdx.x;
    const int cnt = E[(long long)(s + 1) * nblk] - E[(long long)s * nblk];
    const long long lo = (long long)slab_chunk[s] * SLAB_CH + cnt, hi = (long long)slab_chunk[s + 1] * SLAB_CH;
    for (long long j = lo + threadIdx.x; j < hi; j += 64) {
        svals[slab_value_index<SlabOf<T>::G>((int)j)] = T(0);
        scol[j] = 0;
        srow[j] = -1;
        src[j] = -1;
    }
}

// Stable bucketing.  One wave per block of BUILD_BT CSR positions, taken 64 at a time in order; off[s] is the
// slot the block's next position of slab s goes to.  The lanes of one step that share a slab are ranked by
// lane number, so the order of the CSR is kept inside every slab: `nbits` ballots, one per bit of the slab
// number, leave every lane with the mask of the lanes of its slab.  The row of a position is the largest r
// with pos[r] <= p, searched between the rows of the block's first and last position (tile_row = the position
// cut of pos with tiles of BUILD_BT) -- in a copy of that part of pos in LDS when it has at most SCATTER_ROWS
// entries, in global memory otherwise.  The loads of the next 64 positions are issued before the current ones
// are placed.
constexpr int SCATTER_ROWS = 1024;
template <typename T>
__global__ __launch_bounds__(64) void k_slab_scatter(int rows, int nnz, const int *__restrict__ pos,
                                                     const int *__restrict__ crd, const T *__restrict__ vals,
                                                     const int *__restrict__ tile_row, const int *__restrict__ E,
                                                     const int *__restrict__ slab_chunk, int nslabs, int nblk,
                                                     int nbits, T *__restrict__ svals,
                                                     unsigned short *__restrict__ scol, int *__restrict__ srow,
                                                     int *__restrict__ src)
{
    extern __shared__ int off[];                 // [nslabs] next slot of each slab, then [SCATTER_ROWS] row starts
    constexpr int W = SlabOf<T>::W;
    const int b = blockIdx.x, lane = threadIdx.x;
    int *spos = off + nslabs;
    for (int s = lane; s < nslabs; s += WAVE)
        off[s] = slab_chunk[s] * SLAB_CH + (E[(long long)s * nblk + b] - E[(long long)s * nblk]);
    const long long p0 = (long long)b * BUILD_BT;
    const int r_lo = tile_row[b], r_hi = tile_row[b + 1];
    const bool local = r_hi - r_lo < SCATTER_ROWS;          // rows r_lo .. r_hi: at most SCATTER_ROWS of them
    if (local)
        for (int i = lane; i <= r_hi - r_lo; i += WAVE) spos[i] = pos[r_lo + i];
    __syncthreads();
    const unsigned long long below = (1ull << lane) - 1ull;
    int c_next = 0;
    T v_next = 0;
    if (p0 + lane < nnz) { c_next = crd[p0 + lane]; v_next = vals[p0 + lane]; }
    for (int it = 0; it < BUILD_BT / WAVE; ++it) {
        const long long pl = p0 + it * WAVE + lane;
        const bool valid = pl < nnz;
        const int p = valid ? (int)pl : 0;
        const int c = c_next;
        const T v = v_next;
        if (it + 1 < BUILD_BT / WAVE && pl + WAVE < nnz) { c_next = crd[pl + WAVE]; v_next = vals[pl + WAVE]; }
        const int s = valid ? c / W : 0;
        int r = 0;
        if (valid) {
            int lo = r_lo, hi = r_hi;
            if (local) {
                while (lo < hi) {
                    const int mid = lo + ((hi - lo + 1) >> 1);
                    if (spos[mid - r_lo] <= p) lo = mid; else hi = mid - 1;
                }
            } else {
                while (lo < hi) {
                    const int mid = lo + ((hi - lo + 1) >> 1);
                    if (pos[mid] <= p) lo = mid; else hi = mid - 1;
                }
            }
            r = lo;
        }
        // peers = the valid lanes with the same slab number
        unsigned long long peers = __ballot(valid);
        for (int k = 0; k < nbits; ++k) {
            const bool one = (s >> k) & 1;
            const unsigned long long m = __ballot(valid && one);
            peers &= one ? m : ~m;
        }
        int dst = -1;
        if (valid) dst = off[s] + __popcll(peers & below);
        __syncthreads();                                  // one wave: orders the LDS reads before the updates
        if (valid && (peers & below) == 0) off[s] += __popcll(peers);
        __syncthreads();
        if (valid) {
            svals[slab_value_index<SlabOf<T>::G>(dst)] = v;
            scol[dst] = (unsigned short)(c - s * W);
            srow[dst] = r;
            src[dst] = p;
        }
    }
}

// ---- matrices of at most kStageSlabs slabs (8.4 M columns; 4.2 M with fp64 values)
//
// The structure follows from counts per (block of BUILD_BT positions, slab): how many entries, whether one of them belongs to
// the row that enters the block from before (head) and whether one belongs to the row that leaves it (tail).  With these a
// block knows by itself for every entry whether its predecessor and its successor in the slab belong to the same row, i.e.
// where pairs start and end, so every entry is read once, written once and never looked at again.  What is left are
// numbers per start of a pair, not per entry.
// A version that left a row and a source position with every slot (14 bytes written per entry instead of 6), found the
// pairs from them and formed the row lists through two arrays over all entries moved 3.7 GB in 1.28 ms for the power-law matrix
// of 2 M rows and 56.5 M entries; this one moves 1.1 GB.
//
//   k_block_hist   H[b][s] = count | head << 12 | tail << 13
//   k_col_*        E[b][s] = entries of slab s in the blocks before b; totals -> slab_chunk (k_block_bases)
//   k_block_place  values and columns with their end bits to the slots; per start of a pair its slab and rank, in CSR order;
//                  N[b][s] = starts of block b in slab s, N[b][nslabs] = all starts of block b
//   k_col_*        F = the same scan of N; totals -> first pair of every slab (k_block_bases2)
//   k_block_pairs  qidx: pair number = first pair of the slab + F[b][s] + rank
//   k_block_rows   qpos, the position cut of the row lists, chunk_pair, pad slots
constexpr int H_HEAD = 1 << 12, H_TAIL = 1 << 13, H_COUNT = (1 << 12) - 1;
constexpr int BITS_W = BUILD_BT / 64;                 // 64-bit words of a bitmap over a block's positions
static_assert(BUILD_BT <= H_COUNT, "a block's count fits its field");

// Rows that cross the borders of block b: positions below `head` belong to the row that began before the block, positions
// from `tail` on to the row that goes on behind it (tile_row = position cut of pos with tiles of BUILD_BT).
__device__ __forceinline__ void block_borders(const int *__restrict__ pos, const int *__restrict__ tile_row, int b, int nblk,
                                              long long p0, int nvalid, int &head, int &tail)
{
    const int r_lo = tile_row[b], r_hi = tile_row[b + 1];
    head = 0;
    tail = nvalid;
    if (pos[r_lo] < p0) head = (int)min((long long)nvalid, (long long)pos[r_lo + 1] - p0);
    if (b + 1 < nblk && pos[r_hi] < p0 + BUILD_BT) tail = (int)max(0ll, (long long)pos[r_hi] - p0);
}

// A thread takes 8 consecutive positions and adds runs of one slab at once: in the sorted columns of a long row all 64 lanes
// of an instruction that took neighbouring positions would add to one LDS word.
template <int W>
__global__ __launch_bounds__(256) void k_block_hist(int nnz, const int *__restrict__ pos, const int *__restrict__ crd,
                                                    const int *__restrict__ tile_row, int nslabs, int nblk, int vec_ok,
                                                    unsigned short *__restrict__ H)
{
    constexpr int EPT = BUILD_BT / 256;
    static_assert(EPT == 8, "two 16-byte loads per thread");
    __shared__ int hist[kStageSlabs];
    __shared__ unsigned char hflag[kStageSlabs], tflag[kStageSlabs];
    const int b = xcd_tile(blockIdx.x, nblk), tid = threadIdx.x;
    if (b < 0) return;
    hist[tid] = 0;
    hflag[tid] = 0;
    tflag[tid] = 0;
    const long long p0 = (long long)b * BUILD_BT;
    const int nvalid = (int)min((long long)BUILD_BT, (long long)nnz - p0), i0 = tid * EPT;
    int c[EPT];
    if (vec_ok && i0 + EPT <= nvalid) {
#pragma unroll
        for (int g = 0; g < EPT / 4; ++g) {
            const v4i t = ld_stream(reinterpret_cast<const v4i *>(crd + p0 + i0 + 4 * g));
            c[4 * g] = t.x; c[4 * g + 1] = t.y; c[4 * g + 2] = t.z; c[4 * g + 3] = t.w;
        }
    } else {
#pragma unroll
        for (int j = 0; j < EPT; ++j) c[j] = i0 + j < nvalid ? crd[p0 + i0 + j] : 0;
    }
    int head, tail;
    block_borders(pos, tile_row, b, nblk, p0, nvalid, head, tail);
    __syncthreads();
    int cur = -1, n = 0;
#pragma unroll
    for (int j = 0; j < EPT; ++j) {
        const int i = i0 + j;
        if (i < nvalid) {
            const int sl = (int)((unsigned)c[j] / W);
            if (i < head) hflag[sl] = 1;
            if (i >= tail) tflag[sl] = 1;
            if (sl != cur) {
                if (n) atomicAdd(&hist[cur], n);
                cur = sl;
                n = 0;
            }
            ++n;
        }
    }
    if (n) atomicAdd(&hist[cur], n);
    __syncthreads();
    if (tid < nslabs)
        H[(long long)b * nslabs + tid] = (unsigned short)(hist[tid] | (hflag[tid] ? H_HEAD : 0) | (tflag[tid] ? H_TAIL : 0));
}

// ---- exclusive scans down the columns of a matrix M[nblk][S] (the low 12 bits of every entry): sums over chunks of COL_CH
// rows, a scan of every column's chunk sums by one workgroup, then every chunk again on top of its sum.  A thread owns a
// column and every RG-th part of the chunk's rows, so that all accesses run along the rows of M.
constexpr int COL_CH = 64;
__device__ __forceinline__ int col_width(int S) { return S <= 64 ? 64 : (S <= 128 ? 128 : 256); }

template <bool APPLY>
__global__ __launch_bounds__(256) void k_col_chunks(const unsigned short *__restrict__ M, int nblk, int S,
                                                    int *__restrict__ part, int *__restrict__ out)
{
    __shared__ int red[256];
    const int P = col_width(S), RG = 256 / P, rows = COL_CH / RG;
    const int rg = threadIdx.x / P;
    const int b0 = blockIdx.x * COL_CH + rg * rows, b1 = min(min(b0 + rows, (int)(blockIdx.x + 1) * COL_CH), nblk);
    for (int c0 = 0; c0 < S; c0 += P) {                    // more than one round only when S = 257
        const int col = c0 + threadIdx.x % P;
        int sum = 0;
        if (col < S) {
#pragma unroll 8
            for (int b = b0; b < b1; ++b) sum += M[(long long)b * S + col] & H_COUNT;
        }
        __syncthreads();
        red[threadIdx.x] = sum;
        __syncthreads();
        if (!APPLY) {
            if (rg == 0 && col < S) {
                for (int g = 1; g < RG; ++g) sum += red[threadIdx.x + g * P];
                part[(long long)blockIdx.x * S + col] = sum;
            }
        } else if (col < S) {
            int run = part[(long long)blockIdx.x * S + col];
            for (int g = 0; g < rg; ++g) run += red[threadIdx.x % P + g * P];
#pragma unroll 8
            for (int b = b0; b < b1; ++b) {
                out[(long long)b * S + col] = run;
                run += M[(long long)b * S + col] & H_COUNT;
            }
        }
    }
}

// one workgroup per column: exclusive scan of its chunk sums in place, total[col] = their sum
__global__ __launch_bounds__(256) void k_col_scan(int *__restrict__ part, int nparts, int S, int *__restrict__ total)
{
    __shared__ int s_w[4];
    int carry = 0;
    for (int b0 = 0; b0 < nparts; b0 += 256) {
        const int i = b0 + threadIdx.x;
        const int v = i < nparts ? part[(long long)i * S + blockIdx.x] : 0;
        int sum;
        const int inc = block_scan_256(v, s_w, &sum);
        if (i < nparts) part[(long long)i * S + blockIdx.x] = carry + inc - v;
        carry += sum;
    }
    if (threadIdx.x == 0) total[blockIdx.x] = carry;
}

// slab_chunk = exclusive scan of the slabs' sizes in chunks; meta[0] = number of slots
__global__ __launch_bounds__(256) void k_block_bases(const int *__restrict__ total, int nslabs, int *__restrict__ slab_chunk,
                                                     int *__restrict__ meta)
{
    __shared__ int s_w[4];
    const int tid = threadIdx.x;
    const int chunks = tid < nslabs ? (total[tid] + SLAB_CH - 1) / SLAB_CH : 0;
    int sum;
    const int inc = block_scan_256(chunks, s_w, &sum);
    if (tid < nslabs) slab_chunk[tid] = inc - chunks;
    if (tid == 0) {
        slab_chunk[nslabs] = sum;
        meta[0] = sum * SLAB_CH;
    }
}

// slab_pair[s] = first pair of slab s: its starts, and one more pair for its pad slots if it has any (fewer than a chunk, all
// behind the slab's last entry).  meta[1] = pairs, meta[2] = listed pairs.
__global__ __launch_bounds__(256) void k_block_bases2(const int *__restrict__ total, const int *__restrict__ starts, int nslabs,
                                                      const int *__restrict__ slab_chunk, int *__restrict__ slab_pair,
                                                      int *__restrict__ chunk_pair, int *__restrict__ meta)
{
    __shared__ int s_w[4];
    const int tid = threadIdx.x;
    const int pairs = tid < nslabs ? starts[tid] + (total[tid] % SLAB_CH != 0 ? 1 : 0) : 0;
    int sum;
    const int inc = block_scan_256(pairs, s_w, &sum);
    if (tid < nslabs) slab_pair[tid] = inc - pairs;
    if (tid == 0) {
        chunk_pair[slab_chunk[nslabs]] = sum;
        meta[1] = sum;
        meta[2] = starts[nslabs];
    }
}

// A workgroup of four waves per block; wave w takes the w-th quarter, 64 positions per step.  The lanes of a step that share a
// slab are ranked by lane (one ballot per bit of the slab number), a counter per (wave, slab) carries the rank from step to
// step; from the counters every entry gets its place in a staging area in LDS ordered by slab and, inside a slab, by CSR
// position.  Neighbours in the staging area are neighbours in the slab, so starts and ends of pairs are a comparison of row
// ordinals (the number of row starts up to a position: a bitmap and its prefix counts, no search) -- and for the first and
// last entry of a slab's run the question whether the row has entries of this slab in other blocks, answered from H and E.
// The entries leave as runs of consecutive slots; blocks are dealt to the dies in contiguous ranges, so that the runs of
// neighbouring blocks meet in one L2 and reach memory as whole lines.
template <typename T>
__global__ __launch_bounds__(256) void k_block_place(int rows, int nnz, const int *__restrict__ pos, const int *__restrict__ crd,
                                                     const T *__restrict__ vals, const int *__restrict__ tile_row,
                                                     const unsigned short *__restrict__ H, const int *__restrict__ E,
                                                     const int *__restrict__ slab_chunk, int nslabs, int nblk, int nbits,
                                                     T *__restrict__ svals, unsigned short *__restrict__ scol,
                                                     unsigned short *__restrict__ N, int *__restrict__ starts,
                                                     unsigned long long *__restrict__ pbits,
                                                     unsigned short *__restrict__ pbits_pre,
                                                     unsigned long long *__restrict__ chunk_at)
{
    constexpr int W = SlabOf<T>::W, NW = 4, QUART = BUILD_BT / NW, STEPS = QUART / WAVE;
    constexpr int ROWS_WALK = 8 * BUILD_BT;
    __shared__ unsigned short woff[NW][kStageSlabs];   // entries of (wave, slab) so far; later the place of the wave's first one
    __shared__ int lbase[kStageSlabs + 1];             // first staging place of each slab
    __shared__ int gbase[kStageSlabs];                 // slot of a staged entry = gbase[slab] + its place
    __shared__ unsigned short sbase[kStageSlabs];      // starts before the slab's first staging place
    __shared__ T s_val[BUILD_BT];
    __shared__ unsigned s_all[BUILD_BT + 2];           // one entry of no slab on either side
    unsigned *const s_meta = s_all + 1;                // row ordinal (12 bits) | position << 12 (11 bits) | slab << 23
    __shared__ unsigned short s_col[BUILD_BT];
    __shared__ unsigned rowbits[2 * BITS_W], posbits[2 * BITS_W];
    __shared__ unsigned long long startbits[BITS_W], endbits[BITS_W];
    __shared__ int row_pre[BITS_W], pos_pre[BITS_W + 1], start_pre[BITS_W + 1];
    __shared__ int s_w[4];
    const int b = xcd_tile(blockIdx.x, nblk);
    if (b < 0) return;
    const int tid = threadIdx.x, lane = tid & (WAVE - 1);
    const int wave = __builtin_amdgcn_readfirstlane(tid / WAVE);
    const long long p0 = (long long)b * BUILD_BT;
    const int nvalid = (int)min((long long)BUILD_BT, (long long)nnz - p0);

    unsigned c[STEPS];
    T v[STEPS];
    const bool full = nvalid == BUILD_BT;
    {
        const int *const cb = crd + p0 + wave * QUART;
        const T *const vb = vals + p0 + wave * QUART;
        if (full) {
#pragma unroll
            for (int st = 0; st < STEPS; ++st) { c[st] = (unsigned)ld_stream(cb + (st * WAVE + lane)); v[st] = ld_stream(vb + (st * WAVE + lane)); }
        } else {
#pragma unroll
            for (int st = 0; st < STEPS; ++st) {
                const bool valid = wave * QUART + st * WAVE + lane < nvalid;
                c[st] = valid ? (unsigned)cb[st * WAVE + lane] : 0u;
                v[st] = valid ? vb[st * WAVE + lane] : T(0);
            }
        }
    }
    const int r_lo = tile_row[b], r_hi = tile_row[b + 1];
    int h = 0, e = 0;
    if (tid < nslabs) { h = H[(long long)b * nslabs + tid]; e = E[(long long)b * nslabs + tid]; }
    // row starts: the first 256 rows' positions are requested here, ahead of the barrier
    const int p_first = r_lo + 1 + tid <= r_hi ? pos[r_lo + 1 + tid] : 0x7fffffff;
    const int p_lo = pos[r_lo], p_end = r_hi < rows ? pos[r_hi + 1] : nnz;
    for (int i = tid; i < NW * kStageSlabs; i += 256) (&woff[0][0])[i] = 0;
    if (tid < 2 * BITS_W) { rowbits[tid] = 0; posbits[tid] = 0; }
    if (tid == 0) s_all[0] = ~0u;
    for (int i = nvalid + tid; i <= BUILD_BT; i += 256) s_meta[i] = ~0u;
    if (tid < nslabs) gbase[tid] = slab_chunk[tid] * SLAB_CH + e;
    __syncthreads();
    // row starts inside the block; rows that start at its first position need no bit (nothing precedes them here)
    if (r_hi - r_lo <= ROWS_WALK) {
        auto mark = [&](int p) {
            const long long i = (long long)p - p0;
            if (i < nvalid) atomicOr(&rowbits[i >> 5], 1u << (i & 31));
        };
        mark(p_first);
        for (int r = r_lo + 257 + tid; r <= r_hi; r += 256) mark(pos[r]);
    } else {                        // a long run of empty rows: ask for every position instead
        for (int i = tid; i < nvalid; i += 256) {
            const int p = (int)(p0 + i);
            int lo = r_lo, hi = r_hi;
            while (lo < hi) {
                const int mid = lo + ((hi - lo + 1) >> 1);
                if (pos[mid] <= p) lo = mid; else hi = mid - 1;
            }
            if (i > 0 && pos[lo] == p) atomicOr(&rowbits[i >> 5], 1u << (i & 31));
        }
    }
    // Whether the slab's entries of this block continue a pair of an earlier block (the first one belongs to row r_lo, which
    // began in block bp) and whether the last one's row r_hi, which ends in block be, goes on in the slab: requested here,
    // used when the entries are staged.  (Where the block has no such entry the flags of h are clear and the places asked
    // for, held inside the arrays, do not matter.)
    int from = 0, to = 0;
    if (tid < nslabs) {
        const long long bp = p_lo / BUILD_BT, b1 = bp < b ? bp + 1 : b;
        const long long be = max((long long)b, min((long long)nblk - 1, (long long)(p_end > 0 ? p_end - 1 : 0) / BUILD_BT));
        from = (H[bp * nslabs + tid] & H_TAIL) + (e - E[b1 * nslabs + tid]);
        to = (H[be * nslabs + tid] & H_HEAD) + (E[be * nslabs + tid] - e - (h & H_COUNT));
    }
    // rank of every entry among the wave's entries of its slab (a wave touches only its own row of woff; its LDS operations
    // execute in program order)
    int rank[STEPS];
#pragma unroll
    for (int st = 0; st < STEPS; ++st) {
        const int left = nvalid - (wave * QUART + st * WAVE);       // valid lanes of this step (uniform)
        const unsigned long long all = left >= WAVE ? ~0ull : (left > 0 ? (1ull << left) - 1ull : 0ull);
        const unsigned sl = c[st] / W;
        c[st] = (c[st] - sl * W) | (sl << 16);              // column in the slab (15 bits), slab
        unsigned plo = (unsigned)all, phi = (unsigned)(all >> 32);     // peers: the valid lanes with this lane's slab
        if ((__ballot(sl != (unsigned)__builtin_amdgcn_readfirstlane((int)sl)) & all) != 0) {   // sorted columns of a long row: one slab
#pragma unroll
            for (int k = 0; k < 8; ++k) {
                if (k >= nbits) break;
                const int one = __builtin_amdgcn_sbfe((int)sl, k, 1);          // bit k, spread over the word
                const unsigned long long m = __ballot(one != 0);
                plo = __builtin_amdgcn_bitop3_b32(plo, (unsigned)m, (unsigned)one, 0x90);              // a & ~(b ^ c)
                phi = __builtin_amdgcn_bitop3_b32(phi, (unsigned)(m >> 32), (unsigned)one, 0x90);
            }
        }
        const int before = woff[wave][sl];
        const int mine = (int)__builtin_amdgcn_mbcnt_hi(phi, __builtin_amdgcn_mbcnt_lo(plo, 0u));
        rank[st] = before + mine;
        __builtin_amdgcn_wave_barrier();
        if (mine == 0 && lane < left) woff[wave][sl] = (unsigned short)(before + __popc(plo) + __popc(phi));
        __builtin_amdgcn_wave_barrier();
    }
    __syncthreads();
    {
        int n[NW], sum = 0;
#pragma unroll
        for (int w = 0; w < NW; ++w) {
            n[w] = tid < nslabs ? woff[w][tid] : 0;
            sum += n[w];
        }
        int total;
        int o = block_scan_256(sum, s_w, &total) - sum;
        if (tid < nslabs) {
            lbase[tid] = o;
            gbase[tid] -= o;
#pragma unroll
            for (int w = 0; w < NW; ++w) { woff[w][tid] = (unsigned short)o; o += n[w]; }
        }
        if (tid == 0) lbase[nslabs] = total;
        if (wave == 0) {            // row starts before each word of the bitmap
            const int k = lane < BITS_W ? __popc(rowbits[2 * lane]) + __popc(rowbits[2 * lane + 1]) : 0;
            const int inc = wave_scan_add(k);
            if (lane < BITS_W) row_pre[lane] = inc - k;
        }
    }
    __syncthreads();
#pragma unroll
    for (int st = 0; st < STEPS; ++st) {
        const int w = wave * STEPS + st, i = w * WAVE + lane;
        const unsigned lo = (unsigned)rl((int)rowbits[2 * w], 0), hi = (unsigned)rl((int)rowbits[2 * w + 1], 0);
        const unsigned long long word = ((unsigned long long)hi << 32) | lo;
        const int ord = rl(row_pre[w], 0) + (int)(word & 1) + lanes_below(word >> 1);      // row starts up to position i
        if (i < nvalid) {
            const unsigned sl = c[st] >> 16;
            const int li = woff[wave][sl] + rank[st];
            s_val[li] = v[st];
            s_col[li] = (unsigned short)c[st];
            s_meta[li] = (unsigned)ord | ((unsigned)i << 12) | (sl << 23);
        }
    }
    __syncthreads();
    // starts and ends inside the block, as bitmaps over the staging places: an entry starts a pair where slab or row differ
    // from the entry before it, and ends one where the next entry starts one (the places behind the last hold no slab)
    constexpr unsigned KEY = 0xff800fffu;
#pragma unroll
    for (int k = 0; k < BUILD_BT / 256; ++k) {
        const int w = 4 * k + wave, li = w * WAVE + lane;
        const unsigned m = s_meta[li];
        const unsigned long long st = __ballot(((m ^ s_meta[li - 1]) & KEY) != 0), en = __ballot(((m ^ s_meta[li + 1]) & KEY) != 0);
        const int left = nvalid - w * WAVE;                // entries among these places
        if (lane == 0) { startbits[w] = left >= WAVE ? st : (left > 0 ? st & ((1ull << left) - 1ull) : 0ull); endbits[w] = en; }
    }
    __syncthreads();
    // per slab: no start / end where the row's entries of this slab go on in another block, both at the chunks' borders
    if (tid < nslabs && lbase[tid] < lbase[tid + 1]) {
        const int l0 = lbase[tid], l1 = lbase[tid + 1];
        const int g = gbase[tid];
        unsigned *const sb = reinterpret_cast<unsigned *>(startbits), *const eb = reinterpret_cast<unsigned *>(endbits);
        if ((h & H_HEAD) && from > 0) atomicAnd(&sb[l0 >> 5], ~(1u << (l0 & 31)));
        if ((h & H_TAIL) && to > 0) atomicAnd(&eb[(l1 - 1) >> 5], ~(1u << ((l1 - 1) & 31)));
        for (int li = l0 + ((SLAB_CH - ((g + l0) & (SLAB_CH - 1))) & (SLAB_CH - 1)); li <= l1; li += SLAB_CH) {   // slots that begin a chunk
            if (li < l1) atomicOr(&sb[li >> 5], 1u << (li & 31));
            if (li > l0) atomicOr(&eb[(li - 1) >> 5], 1u << ((li - 1) & 31));
        }
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < BUILD_BT / 256; ++k) {
        const int w = 4 * k + wave, li = w * WAVE + lane;
        if (li < nvalid) {
            const unsigned m = s_meta[li];
            const int dst = gbase[m >> 23] + li;
            const unsigned word = lane < 32 ? (unsigned)endbits[w] : (unsigned)(endbits[w] >> 32);
            svals[slab_value_index<SlabOf<T>::G>(dst)] = s_val[li];
            scol[dst] = (unsigned short)(s_col[li] | (((word >> (lane & 31)) & 1u) << 15));
            const unsigned sw = lane < 32 ? (unsigned)startbits[w] : (unsigned)(startbits[w] >> 32);
            const unsigned i = (m >> 12) & (BUILD_BT - 1);
            if ((sw >> (lane & 31)) & 1u) atomicOr(&posbits[i >> 5], 1u << (i & 31));
        }
    }
    __syncthreads();
    if (wave == 0) {
        const int k = lane < BITS_W ? __popcll(startbits[lane]) : 0;
        const int inc = wave_scan_add(k);
        if (lane <= BITS_W) start_pre[lane] = inc - k;
    } else if (wave == 1) {
        const unsigned lo = lane < BITS_W ? posbits[2 * lane] : 0, hi = lane < BITS_W ? posbits[2 * lane + 1] : 0;
        const int k = __popc(lo) + __popc(hi);
        const int inc = wave_scan_add(k);
        if (lane < BITS_W) {
            pos_pre[lane] = inc - k;
            pbits[(long long)b * BITS_W + lane] = ((unsigned long long)hi << 32) | lo;
            pbits_pre[(long long)b * BITS_W + lane] = (unsigned short)(inc - k);
        }
    }
    __syncthreads();
    auto starts_before = [&](int li) {                 // starts at staging places below li
        const int w = li >> 6;
        return li >= BUILD_BT ? start_pre[BITS_W] : start_pre[w] + __popcll(startbits[w] & ((1ull << (li & 63)) - 1ull));
    };
    if (tid < nslabs) {
        const int n0 = starts_before(lbase[tid]), n1 = starts_before(lbase[tid + 1]);
        sbase[tid] = (unsigned short)n0;
        N[(long long)b * (nslabs + 1) + tid] = (unsigned short)(n1 - n0);
    }
    if (tid == 0) N[(long long)b * (nslabs + 1) + nslabs] = (unsigned short)start_pre[BITS_W];
    __syncthreads();
#pragma unroll
    for (int k = 0; k < BUILD_BT / 256; ++k) {
        const int w = 4 * k + wave;
        const unsigned long long word = startbits[w];
        const int nth_start = start_pre[w] + lanes_below(word);
        if ((word >> lane) & 1ull) {
            const int li = tid + 256 * k;
            const unsigned m = s_meta[li], sl = m >> 23;
            const int dst = gbase[sl] + li;
            const unsigned e = (sl << 16) | (unsigned)(nth_start - sbase[sl]);
            const unsigned i = (m >> 12) & (BUILD_BT - 1), iw = i >> 6;
            const unsigned long long pw = ((unsigned long long)posbits[2 * iw + 1] << 32) | posbits[2 * iw];
            starts[p0 + pos_pre[iw] + __popcll(pw & ((1ull << (i & 63)) - 1ull))] = (int)e;
            if ((dst & (SLAB_CH - 1)) == 0) chunk_at[dst / SLAB_CH] = ((unsigned long long)b << 32) | e;
        }
    }
}

// qidx: a wave per block writes the pair numbers of the block's starts, in CSR order
__global__ __launch_bounds__(256) void k_block_pairs(const unsigned short *__restrict__ N, const int *__restrict__ F,
                                                     const int *__restrict__ slab_pair, const int *__restrict__ starts, int nslabs,
                                                     int nblk, int *__restrict__ qidx)
{
    const int g = xcd_tile(blockIdx.x, (nblk + 3) / 4), lane = threadIdx.x & (WAVE - 1);
    const int b = g * 4 + __builtin_amdgcn_readfirstlane(threadIdx.x / WAVE);
    if (g < 0 || b >= nblk) return;
    const long long row = (long long)b * (nslabs + 1);
    const int n = N[row + nslabs], q0 = F[row + nslabs];
    for (int k0 = lane; k0 < n; k0 += 8 * WAVE) {          // 337 starts per block on average: one round, all loads in flight
        int e[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) e[u] = k0 + u * WAVE < n ? ld_stream(starts + (long long)b * BUILD_BT + k0 + u * WAVE) : 0;
#pragma unroll
        for (int u = 0; u < 8; ++u) e[u] = slab_pair[e[u] >> 16] + F[row + (e[u] >> 16)] + (e[u] & 0xffff);
#pragma unroll
        for (int u = 0; u < 8; ++u)
            if (k0 + u * WAVE < n) qidx[q0 + k0 + u * WAVE] = e[u];
    }
}

// Thread g: row g's first listed pair (the starts before pos[g]: the block's count plus the bits below it) and the table
// entries of the row-list tiles that begin in the row; chunk g's first pair; pad slot g % 512 of slab g / 512.
template <typename T>
__global__ __launch_bounds__(256) void k_block_rows(int rows, int nnz, const int *__restrict__ pos, const int *__restrict__ F,
                                                    const unsigned long long *__restrict__ pbits,
                                                    const unsigned short *__restrict__ pbits_pre,
                                                    const unsigned long long *__restrict__ chunk_at,
                                                    const int *__restrict__ total, const int *__restrict__ slab_pair,
                                                    const int *__restrict__ slab_chunk, int nslabs, int tile,
                                                    const int *__restrict__ meta, T *__restrict__ svals,
                                                    unsigned short *__restrict__ scol, int *__restrict__ chunk_pair,
                                                    int *__restrict__ qpos, int *__restrict__ qtile_row)
{
    const long long g = (long long)blockIdx.x * 256 + threadIdx.x;
    const int lane = threadIdx.x & (WAVE - 1);
    const int nq = meta[2], S1 = nslabs + 1;
    auto listed = [&](int p) -> int {                  // starts at CSR positions below p
        if (p >= nnz) return nq;
        const long long b = p / BUILD_BT;
        const int i = p % BUILD_BT;
        const long long w = b * BITS_W + (i >> 6);
        return F[b * S1 + nslabs] + pbits_pre[w] + __popcll(pbits[w] & ((1ull << (i & 63)) - 1ull));
    };
    int t_lo = 0, t_hi = -1;
    if (g <= rows) {
        const int q = listed(pos[g]);
        qpos[g] = q;
        if (g < rows) {
            const int q1 = listed(pos[g + 1]);
            if (q1 > q) {
                t_lo = (int)(((long long)q + tile - 1) / tile);
                t_hi = (q1 - 1) / tile;
            }
        } else qtile_row[((long long)nq + tile - 1) / tile] = rows;
    }
    const int n = t_hi - t_lo + 1;
    if (n > 0 && n <= 16)
        for (int t = t_lo; t <= t_hi; ++t) qtile_row[t] = (int)g;
    unsigned long long big = __ballot(n > 16);
    while (big) {
        const int src = __ffsll((long long)big) - 1;
        big &= big - 1;
        const int lo = __shfl(t_lo, src, WAVE), hi = __shfl(t_hi, src, WAVE), row = __shfl((int)g, src, WAVE);
        for (int t = lo + lane; t <= hi; t += WAVE) qtile_row[t] = row;
    }
    if (g < meta[0] / SLAB_CH) {
        const unsigned long long a = chunk_at[g];
        const int sl = (int)((a >> 16) & 0xffff);
        chunk_pair[g] = slab_pair[sl] + F[(long long)(a >> 32) * S1 + sl] + (int)(a & 0xffff);
    }
    if (g < (long long)nslabs * SLAB_CH) {
        const int sl = (int)(g / SLAB_CH);
        const long long hi = (long long)slab_chunk[sl + 1] * SLAB_CH;
        const long long j = (long long)slab_chunk[sl] * SLAB_CH + total[sl] + g % SLAB_CH;
        if (j < hi) {               // value 0, column 0; the last one ends the pads' pair
            svals[slab_value_index<SlabOf<T>::G>((int)j)] = T(0);
            scol[j] = j + 1 == hi ? 0x8000u : 0u;
        }
    }
}

// ---- more slabs: a row and a source position per slot, pairs found from them
// Pairs.  One wave per chunk; slot j = chunk * CH + it * 64 + lane (it = 0 .. 7), so that the rows of the slots are read
// with full-width loads.  A slot starts a pair when it is the chunk's first or its row differs from the row of the slot
// before it (the lane below, or lane 63 of the round before); m[it] = the ballot of the starts of round it.
constexpr int SLAB_ROUNDS = SLAB_CH / WAVE;
__device__ __forceinline__ void chunk_starts(const int *__restrict__ srow, long long base, int lane,
                                             unsigned long long (&m)[SLAB_ROUNDS], int (&r)[SLAB_ROUNDS])
{
#pragma unroll
    for (int it = 0; it < SLAB_ROUNDS; ++it) r[it] = srow[base + it * WAVE + lane];
    int last = 0;
#pragma unroll
    for (int it = 0; it < SLAB_ROUNDS; ++it) {
        int prev = __shfl_up(r[it], 1, WAVE);
        if (lane == 0) prev = last;
        m[it] = __ballot((it == 0 && lane == 0) || r[it] != prev);
        last = rl(r[it], WAVE - 1);
    }
}

// cnt[c] = number of pairs of chunk c for c < nslots / CH (nslots = meta[0]), 0 for the entries up to `nmaxchunks`
// (the array is scanned over its whole length: its exclusive scan is chunk_pair).
__global__ __launch_bounds__(256) void k_slab_count(const int *__restrict__ meta, const int *__restrict__ srow,
                                                    int nmaxchunks, int *__restrict__ cnt)
{
    const int lane = threadIdx.x & (WAVE - 1);
    const int c = blockIdx.x * 4 + __builtin_amdgcn_readfirstlane(threadIdx.x / WAVE);
    if (c > nmaxchunks) return;
    const int nch = meta[0] / SLAB_CH;
    int total = 0;
    if (c < nch) {
        unsigned long long m[SLAB_ROUNDS];
        int r[SLAB_ROUNDS];
        chunk_starts(srow, (long long)c * SLAB_CH, lane, m, r);
#pragma unroll
        for (int it = 0; it < SLAB_ROUNDS; ++it) total += __popcll(m[it]);
    }
    if (lane == 0) cnt[c] = total;
}

// With chunk_pair = the exclusive scan of cnt: sets the end-of-pair bit of every pair's last slot (the slot before a
// start, and the chunk's last slot) and, for the first slot of every pair of a real row, leaves the pair's number + 1 at
// the CSR position the slot came from (pair_at, zero elsewhere), from which the row lists are formed.
// meta[1] = number of pairs.
__global__ __launch_bounds__(256) void k_slab_close(const int *__restrict__ meta_in, const int *__restrict__ srow,
                                                    const int *__restrict__ src, const int *__restrict__ chunk_pair,
                                                    unsigned short *__restrict__ scol, int *__restrict__ pair_at,
                                                    int *__restrict__ meta)
{
    const int lane = threadIdx.x & (WAVE - 1);
    const int c = blockIdx.x * 4 + __builtin_amdgcn_readfirstlane(threadIdx.x / WAVE);
    const int nch = meta_in[0] / SLAB_CH;
    if (c >= nch) return;
    const long long base = (long long)c * SLAB_CH;
    unsigned long long m[SLAB_ROUNDS];
    int r[SLAB_ROUNDS];
    chunk_starts(srow, base, lane, m, r);
    const int cp = chunk_pair[c];
    int before = 0;                                         // pairs of the chunk that start in earlier rounds
#pragma unroll
    for (int it = 0; it < SLAB_ROUNDS; ++it) {
        const long long j = base + it * WAVE + lane;
        const bool start = (m[it] >> lane) & 1ull;
        const bool end = lane < WAVE - 1 ? (m[it] >> (lane + 1)) & 1ull
                                         : (it < SLAB_ROUNDS - 1 ? m[it + 1 < SLAB_ROUNDS ? it + 1 : it] & 1ull : 1ull);
        if (end) scol[j] = (unsigned short)(scol[j] | 0x8000u);
        if (start && r[it] >= 0) {
            const int mine = cp + before + __popcll(m[it] & (~0ull >> (WAVE - 1 - lane))) - 1;     // this slot's pair
            pair_at[src[j]] = mine + 1;
        }
        before += __popcll(m[it]);
    }
    if (c == nch - 1 && lane == 0) meta[1] = chunk_pair[nch];
}

// R = exclusive scan of (pair_at != 0) over nnz + 1 entries: R[p] = number of pairs whose first slot comes from a CSR
// position below p.  Rows list their pairs in that order: qpos[r] = R[pos[r]], qidx[R[p]] = pair_at[p] - 1.
// meta[2] = number of listed pairs.
__global__ __launch_bounds__(256) void k_slab_rows(int rows, int nnz, const int *__restrict__ pos,
                                                   const int *__restrict__ R, const int *__restrict__ pair_at,
                                                   int *__restrict__ qpos, int *__restrict__ qidx,
                                                   int *__restrict__ meta)
{
    const long long g = (long long)blockIdx.x * 256 + threadIdx.x;
    if (g < nnz) {
        const int a = R[g];
        if (R[g + 1] != a) qidx[a] = pair_at[g] - 1;
    }
    if (g <= rows) qpos[g] = R[pos[g]];
    if (g == 0) meta[2] = R[nnz];
}

__global__ __launch_bounds__(256) void k_fill_int(int *__restrict__ p, long long n, int v)
{
    long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    const long long stride = (long long)gridDim.x * blockDim.x;
    for (; i < n; i += stride) p[i] = v;
}

hipError_t launch_fill_int(int32_t *p, int64_t n, int32_t v, hipStream_t s)
{
    if (n <= 0) return hipSuccess;
    int64_t blocks = (n + 255) / 256;
    if (blocks > 65536) blocks = 65536;
    PSK_LAUNCH(k_fill_int, dim3((unsigned)blocks), dim3(256), 0, s, p, (long long)n, v);
    return take_launch_status();
}

SlabBuildSpace carve_slab_build(void *base, int64_t rows, int64_t cols, int64_t nnz, int32_t W)
{
    (void)rows;
    SlabBuildSpace w;
    const int64_t S = (cols + W - 1) / W;
    const int64_t nblk = (nnz + BUILD_BT - 1) / BUILD_BT;
    const int64_t nmax = slab_max_slots(cols, nnz, W);
    char *p = static_cast<char *>(base);
    size_t o = 0;
    auto take = [&](size_t bytes) { char *q = p + o; o += align256(bytes); return q; };
    w = SlabBuildSpace{};
    w.meta = reinterpret_cast<int32_t *>(take(256));
    w.tile_row = reinterpret_cast<int32_t *>(take((size_t)(nblk + 1) * 4));
    if (S <= kStageSlabs) {
        const size_t S1 = (size_t)S + 1;
        w.total = reinterpret_cast<int32_t *>(take(3 * S1 * 4));
        w.part = reinterpret_cast<int32_t *>(take((size_t)((nblk + COL_CH - 1) / COL_CH) * S1 * 4));
        w.H16 = reinterpret_cast<uint16_t *>(take((size_t)nblk * (size_t)S * 2));
        w.N16 = reinterpret_cast<uint16_t *>(take((size_t)nblk * S1 * 2));
        w.H = reinterpret_cast<int32_t *>(take((size_t)nblk * S1 * 4));
        w.src = reinterpret_cast<int32_t *>(take((size_t)(nnz + 1) * 4));                 // starts of pairs, per block
        w.pbits = reinterpret_cast<unsigned long long *>(take((size_t)nblk * BITS_W * 8));
        w.pbits_pre = reinterpret_cast<uint16_t *>(take((size_t)nblk * BITS_W * 2));
        w.chunk_at = reinterpret_cast<unsigned long long *>(take((size_t)(nmax / SLAB_CH + 1) * 8));
        w.bytes = o;
        return w;
    }
    w.H = reinterpret_cast<int32_t *>(take((size_t)(S * nblk + 1) * 4));
    w.srow = reinterpret_cast<int32_t *>(take((size_t)(nmax + 1) * 4));
    w.src = reinterpret_cast<int32_t *>(take((size_t)(nmax + 1) * 4));
    w.F = reinterpret_cast<int32_t *>(take((size_t)(nmax / SLAB_CH + 2) * 4));       // pairs per chunk
    w.mark = reinterpret_cast<int32_t *>(take((size_t)(nnz + 1) * 4));
    w.pair_at = reinterpret_cast<int32_t *>(take((size_t)(nnz + 1) * 4));
    size_t tmp = scan_tmp_ints(S * nblk + 1);
    if (scan_tmp_ints(nnz + 1) > tmp) tmp = scan_tmp_ints(nnz + 1);
    w.scan_tmp = reinterpret_cast<int32_t *>(take(tmp * 4));
    w.bytes = o;
    return w;
}

// Enqueues the whole analysis on `s`.  When it has run, meta[0..2] = {slots, pairs, listed pairs}.  qtile_row (the position
// cut of the row lists) is written for at most kStageSlabs slabs; with more the caller makes it once it knows their number.
template <typename T>
static hipError_t launch_slab_build_t(int32_t rows, int32_t cols, int32_t nnz, const int32_t *pos, const int32_t *crd,
                                      const T *vals, const SlabBuildSpace &w, T *svals, uint16_t *scol,
                                      int32_t *chunk_pair, int32_t *slab_chunk, int32_t *qpos, int32_t *qidx,
                                      int32_t qtile, int32_t *qtile_row, hipStream_t s)
{
    constexpr int W = SlabOf<T>::W;
    const int S = (int)(((int64_t)cols + W - 1) / W);
    const int nblk = (int)(((int64_t)nnz + BUILD_BT - 1) / BUILD_BT);
    const int64_t nmax = slab_max_slots(cols, nnz, W);
    unsigned short *scol_d = reinterpret_cast<unsigned short *>(scol);
    hipError_t e = launch_partition(rows, nnz, pos, BUILD_BT, 0, w.tile_row, s);
    if (e != hipSuccess) return e;
    int nbits = 0;                                  // bits of a slab number
    while ((1 << nbits) < S) ++nbits;
    if (S <= kStageSlabs) {
        const int S1 = S + 1, nparts = (nblk + COL_CH - 1) / COL_CH, grid = xcd_grid(nblk);
        int32_t *total = w.total, *starts_total = w.total + S1, *slab_pair = w.total + 2 * S1, *E = w.H, *F = w.H;
        const int vec_ok = (reinterpret_cast<uintptr_t>(crd) & 15) == 0;
        PSK_LAUNCH(k_block_hist<W>, dim3(grid), dim3(256), 0, s, nnz, pos, crd, w.tile_row, S, nblk, vec_ok, w.H16);
        PSK_LAUNCH(k_col_chunks<false>, dim3(nparts), dim3(256), 0, s, w.H16, nblk, S, w.part, E);
        PSK_LAUNCH(k_col_scan, dim3(S), dim3(256), 0, s, w.part, nparts, S, total);
        PSK_LAUNCH(k_col_chunks<true>, dim3(nparts), dim3(256), 0, s, w.H16, nblk, S, w.part, E);
        PSK_LAUNCH(k_block_bases, dim3(1), dim3(256), 0, s, total, S, slab_chunk, w.meta);
        PSK_LAUNCH(k_block_place<T>, dim3(grid), dim3(256), 0, s, rows, nnz, pos, crd, vals, w.tile_row, w.H16, E, slab_chunk, S, nblk,
                   nbits, svals, scol_d, w.N16, w.src, w.pbits, w.pbits_pre, w.chunk_at);
        PSK_LAUNCH(k_col_chunks<false>, dim3(nparts), dim3(256), 0, s, w.N16, nblk, S1, w.part, F);
        PSK_LAUNCH(k_col_scan, dim3(S1), dim3(256), 0, s, w.part, nparts, S1, starts_total);
        PSK_LAUNCH(k_col_chunks<true>, dim3(nparts), dim3(256), 0, s, w.N16, nblk, S1, w.part, F);
        PSK_LAUNCH(k_block_bases2, dim3(1), dim3(256), 0, s, total, starts_total, S, slab_chunk, slab_pair, chunk_pair, w.meta);
        PSK_LAUNCH(k_block_pairs, dim3(xcd_grid((nblk + 3) / 4)), dim3(256), 0, s, w.N16, F, slab_pair, w.src, S, nblk, qidx);
        int64_t span = (int64_t)rows + 1;
        if (nmax / SLAB_CH > span) span = nmax / SLAB_CH;
        if ((int64_t)S * SLAB_CH > span) span = (int64_t)S * SLAB_CH;
        PSK_LAUNCH(k_block_rows<T>, dim3((unsigned)((span + 255) / 256)), dim3(256), 0, s, rows, nnz, pos, F, w.pbits, w.pbits_pre,
                   w.chunk_at, total, slab_pair, slab_chunk, S, qtile, w.meta, svals, scol_d, chunk_pair, qpos, qtile_row);
        return take_launch_status();
    }
    const size_t lds = (size_t)S * 4;
    PSK_LAUNCH(k_slab_hist, dim3(nblk), dim3(256), (unsigned)lds, s, nnz, crd, W, S, nblk, w.H);
    PSK_LAUNCH(k_fill_int, dim3(1), dim3(64), 0, s, w.H + (long long)S * nblk, 1ll, 0);      // the scan's total slot
    launch_scan(w.H, w.H, (int64_t)S * nblk + 1, w.scan_tmp, false, s);
    PSK_LAUNCH(k_slab_bases, dim3(1), dim3(256), 0, s, w.H, S, nblk, slab_chunk, w.meta);
    PSK_LAUNCH(k_slab_pads<T>, dim3(S), dim3(64), 0, s, w.H, nblk, slab_chunk, svals, scol_d, w.srow, w.src);
    PSK_LAUNCH(k_slab_scatter<T>, dim3(nblk), dim3(64), (unsigned)(lds + SCATTER_ROWS * 4), s, rows, nnz, pos, crd, vals,
               w.tile_row, w.H, slab_chunk, S, nblk, nbits, svals, scol_d, w.srow, w.src);
    const int nmaxchunks = (int)(nmax / SLAB_CH);
    PSK_LAUNCH(k_slab_count, dim3((unsigned)(nmaxchunks / 4 + 1)), dim3(256), 0, s, w.meta, w.srow, nmaxchunks, w.F);
    launch_scan(w.F, chunk_pair, (int64_t)nmaxchunks + 1, w.scan_tmp, false, s);
    {
        int64_t blocks = ((int64_t)nnz + 1 + 255) / 256;
        if (blocks > 65536) blocks = 65536;
        PSK_LAUNCH(k_fill_int, dim3((unsigned)blocks), dim3(256), 0, s, w.pair_at, (long long)nnz + 1, 0);
    }
    PSK_LAUNCH(k_slab_close, dim3((unsigned)(nmaxchunks / 4 + 1)), dim3(256), 0, s, w.meta, w.srow, w.src, chunk_pair,
               scol_d, w.pair_at, w.meta);
    launch_scan(w.pair_at, w.mark, (int64_t)nnz + 1, w.scan_tmp, true, s);
    const int64_t span = ((int64_t)nnz > (int64_t)rows + 1 ? (int64_t)nnz : (int64_t)rows + 1);
    PSK_LAUNCH(k_slab_rows, dim3((unsigned)((span + 255) / 256)), dim3(256), 0, s, rows, nnz, pos, w.mark, w.pair_at,
               qpos, qidx, w.meta);
    return take_launch_status();
}

hipError_t launch_slab_build(int32_t rows, int32_t cols, int32_t nnz, const int32_t *pos, const int32_t *crd,
                             const float *vals, const SlabBuildSpace &w, float *svals, uint16_t *scol,
                             int32_t *chunk_pair, int32_t *slab_chunk, int32_t *qpos, int32_t *qidx, int32_t qtile,
                             int32_t *qtile_row, hipStream_t s)
{
    return launch_slab_build_t<float>(rows, cols, nnz, pos, crd, vals, w, svals, scol, chunk_pair, slab_chunk, qpos, qidx, qtile, qtile_row, s);
}

hipError_t launch_slab_build_f64(int32_t rows, int32_t cols, int32_t nnz, const int32_t *pos, const int32_t *crd,
                                 const double *vals, const SlabBuildSpace &w, double *svals, uint16_t *scol,
                                 int32_t *chunk_pair, int32_t *slab_chunk, int32_t *qpos, int32_t *qidx, int32_t qtile,
                             int32_t *qtile_row, hipStream_t s)
{
    return launch_slab_build_t<double>(rows, cols, nnz, pos, crd, vals, w, svals, scol, chunk_pair, slab_chunk, qpos, qidx, qtile, qtile_row, s);
}

#ifdef PSK_CU_TRACE
hipError_t cu_trace_set_slab(void *buf, unsigned records) { return cu_trace_set_here(buf, records); }
#endif

}  // namespace psk
