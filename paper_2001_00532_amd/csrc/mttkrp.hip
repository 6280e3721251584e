// MTTKRP on a three-level compressed tensor in position space (appendix "MTTKRP on a GPU"):
//     A(i,j) = B(i,k,l) * C(k,j) * D(l,j)
// Schedule: the k and l loops are fused, then i with them; the fused loop runs over the positions of
// B's leaf level, split into tiles (workgroups) and wave chunks; j is split over the lanes; the loop
// over a wave's positions is innermost.  Section 3: a position loop keeps track of every coordinate
// above the cut the same way it tracks the row of a CSR matrix -- here two levels, fiber and slice.
#include "psk_dev.h"
#include "psk_internal.h"

namespace psk {

// Largest i in [0, n] with a[i] <= target (a[0] <= target taken for granted), by L neighbouring lanes: a round probes L places at
// equal steps and leaves one L + 1-th.  Every lane of the L gets the result.
template <int L>
__device__ __forceinline__ int lanes_search(const int *__restrict__ a, int n, int target)
{
    const unsigned lane = threadIdx.x & (WAVE - 1), sub = lane % L;
    unsigned lo = 0, hi = (unsigned)n;
    if constexpr (L == 1) {                       // (one by one, without the ballots: 366 542 entries, 2.3 M fibers 17.3 -> 13.2 us)
        while (lo < hi) {
            const unsigned mid = lo + ((hi - lo + 1) >> 1);
            if (a[mid] <= target) lo = mid;
            else hi = mid - 1;
        }
    }
    while (__ballot(lo < hi)) {
        const unsigned step = (hi - lo) / (L + 1) + 1, i = lo + (sub + 1) * step;
        const bool below = lo < hi && i <= hi && a[i <= hi ? i : hi] <= target;
        const unsigned long long all = __ballot(below);
        const unsigned c = (unsigned)__popcll(L == WAVE ? all : (all >> (lane - sub)) & ((1ull << (L % WAVE)) - 1ull));
        if (lo < hi) {
            lo += c * step;
            hi = min(hi, lo + step - 1);
        }
    }
    return (int)lo;
}

// tile_fiber[t] = largest q in [0, nfibers] with pos_l[q] <= min(t*tile, nnz); tile_slice[t] = largest s in
// [0, nslices] with pos_k[s] <= tile_fiber[t]: two chained searches (Section 6.2), L lanes per entry.  Bound by the chain of dependent
// loads: 4 M fibers in 500 000 slices take 41 of them one by one (a lane per entry); see the launcher for what more lanes give.
template <int L>
__global__ __launch_bounds__(256) void k_partition_csf3(int nslices, int nfibers, int nnz,
                                                        const int *__restrict__ pos_k,
                                                        const int *__restrict__ pos_l, int tile, int ntiles,
                                                        int *__restrict__ tile_slice,
                                                        int *__restrict__ tile_fiber)
{
    const long long g = ((long long)blockIdx.x * 256 + threadIdx.x) / L;
    const int t = g < ntiles ? (int)g : ntiles;             // (lanes behind the last entry repeat it: the ballots need whole waves)
    const long long first = (long long)t * tile;
    const int target = first < nnz ? (int)first : nnz;
    const int q = lanes_search<L>(pos_l, nfibers, target);
    const int s = lanes_search<L>(pos_k, nslices, q);
    if (threadIdx.x % L == 0 && g <= ntiles) {
        tile_fiber[t] = q;
        tile_slice[t] = s;
    }
}

hipError_t launch_partition_csf3(int32_t nslices, int32_t nfibers, int32_t nnz, const int32_t *pos_k,
                                 const int32_t *pos_l, int32_t tile, int32_t *tile_slice, int32_t *tile_fiber,
                                 hipStream_t s)
{
    const int ntiles = nnz <= 0 ? 0 : (int)(((int64_t)nnz + tile - 1) / tile);
#define PSK_GO(L)                                                                                                 \
    PSK_LAUNCH(k_partition_csf3<L>, dim3((unsigned)(((int64_t)(ntiles + 1) * L + 255) / 256)), dim3(256), 0, s, nslices, nfibers, \
               nnz, pos_k, pos_l, tile, ntiles, tile_slice, tile_fiber)
    // 666 tiles, 120 000 fibers 8.6 us with a lane per entry, 6.7 with 64 (16: 8.2); 2 843 and 500 000 9.8, 6.9; 9 096 and 1.6 M 10.5, 7.5;  22 788
    // and 4 M 11.0, 17 (4 lanes 8.4, 8 9.2);  72 766 and 1.6 M 10.5, 36 (4: 7.2);  182 297 and 4 M 14.0 (4: 16.2; 1 with the ballots of the others 17)
    if (ntiles <= 12000) PSK_GO(64);
    else if (ntiles <= 100000) PSK_GO(4);
    else PSK_GO(1);
#undef PSK_GO
    return take_launch_status();
}

// One workgroup (4 waves) per tile of T leaf positions and per chunk of 64/G columns.
//
// Tile metadata in LDS: sflag[i] = s if leaf position i is the last leaf of slice s (slices play the role
// the rows play in SpMM; a slice's leaves are pos_l[pos_k[s]] .. pos_l[pos_k[s+1]]), and sk[i] = the mode-k
// coordinate k of the fiber that owns leaf i, stored as ~k on the fiber's last leaf in the tile (filled fiber
// by fiber from the tile's window of pos_l; fibers with >= LONGF leaves in the tile are filled by a whole
// wave).  Slices without leaves that fall into the
// tile's write range get zero rows.
// A wave walks its leaves 64 at a time: l, k, flag and value are loaded one per lane and broadcast with
// v_readlane, so that the rows D[l,:] and C[k,:] are wave-uniform, contiguous loads; U rows of D are
// requested before the first multiply.  Within a fiber the product is regrouped by distributivity,
// A(i,:) += C(k,:) * sum_l B(i,k,l) D(l,:), so the C row is requested once, where the fiber's partial sum
// closes (its last leaf in the tile, or the wave's last leaf), not once per leaf: a cache hit between every
// two misses of the D gather costs bandwidth, because the vector memory pipeline returns in order.
// Segments, records, carries: as in the SpMM kernel (the first and last open segments of each wave are
// chained by wave 0; a chain whose slice began before the tile becomes the tile's carry record).
// A lane owns VEC adjacent columns.  G > 1 (VEC = 1, narrow factor matrices, j <= 64/G): the wave is split into G groups of 64/G lanes and in one
// step the groups take G consecutive leaves, so that one load instruction fetches G rows of D.  A lane keeps
// its group's share of the open fiber and of the open slice; a fiber end multiplies every share by the C row
// (no exchange needed: the product distributes over the shares), a slice end adds the shares across groups.
template <int VEC, int G>
__global__ __launch_bounds__(256) void k_mttkrp_pos(int nslices, int nnz, const int *__restrict__ crd_i,
                                                    const int *__restrict__ pos_k,
                                                    const int *__restrict__ crd_k,
                                                    const int *__restrict__ pos_l,
                                                    const int *__restrict__ crd_l,
                                                    const float *__restrict__ vals,
                                                    const float *__restrict__ C, long long ldc,
                                                    const float *__restrict__ D, long long ldd, int jdim,
                                                    float *__restrict__ A, long long lda,
                                                    const int *__restrict__ tile_slice,
                                                    const int *__restrict__ tile_fiber,
                                                    int *__restrict__ carry_row,
                                                    float *__restrict__ carry_val, int ntiles, int T)
{
    static_assert(VEC == 1 || G == 1, "groups of lanes own single columns");
    constexpr int THREADS = 256, NW = THREADS / WAVE, GW = WAVE / G, KW = GW * VEC, LONGF = 32;
    constexpr int U = G > 1 ? 4 : 8;              // steps whose D rows are in flight together
    extern __shared__ int smeta[];                // sflag[T], sk[T], long-fiber queue [3 * T / LONGF]
    int *sflag = smeta, *sk = smeta + T, *slong = smeta + 2 * T;
    __shared__ float srec[2 * NW][KW];
    __shared__ int srec_row[2 * NW];              // -2 unused, -1 open segment, >= 0 slice that ended
    __shared__ int nlong;

    const int t = xcd_tile(blockIdx.x, ntiles);
    if (t < 0) return;
    const int tid = threadIdx.x, lane = tid & (WAVE - 1);
    const int wave = __builtin_amdgcn_readfirstlane(tid / WAVE);   // tells the compiler it is uniform
    const int t0 = t * T;
    const int cnt = (nnz - t0 < T) ? nnz - t0 : T;
    const int t1 = t0 + cnt;
    const int g = lane / GW, gl = lane % GW;      // group of the lane, lane inside the group (G = 1: 0, lane)
    const int col = blockIdx.y * KW + gl * VEC;
    const bool active = col < jdim;
    const bool writer = active && g == 0;         // group 0 stores on behalf of the wave
    const int lcol = active ? col : 0;            // lanes past the last column load column 0 and store nothing

    for (int i = tid; i < T; i += THREADS) { sflag[i] = -1; sk[i] = 0; }
    if (tid < 2 * NW) srec_row[tid] = -2;
    if (tid == 0) nlong = 0;

    const int r0 = tile_slice[t], r1 = tile_slice[t + 1];
    const int q0 = tile_fiber[t], q1 = tile_fiber[t + 1];
    const int leaf_r0 = pos_l[pos_k[r0]], leaf_r1 = pos_l[pos_k[r1]];   // first leaf of slices r0, r1
    const bool has_carry = (t > 0) && (leaf_r0 < t0);
    const int rbeg = (t == 0) ? 0 : r0;
    const bool straddle = leaf_r1 != t1;          // slice r1 continues into the next tile
    const int rend = straddle ? r1 + 1 : r1;
    const int qend = (pos_l[q1] != t1) ? q1 + 1 : q1;   // fibers with leaves in this tile: q0 .. qend-1
    if (tid == 0 && blockIdx.y == 0 && !has_carry) carry_row[t] = -1;
    __syncthreads();

    // ---- slice ends of this tile, zero rows for slices without leaves
    for (int rb = rbeg + wave * WAVE; rb < rend; rb += THREADS) {
        const int r = rb + lane;
        const bool valid = r < rend;
        const int ps = valid ? pos_l[pos_k[r]] : 0, pe = valid ? pos_l[pos_k[r + 1]] : 1;
        if (valid && pe > ps) {
            const int e = pe - 1 - t0;
            if (e >= 0 && e < cnt) sflag[e] = r;
        }
        unsigned long long empty = __ballot(valid && pe == ps);
        while (empty) {
            const int j = __ffsll((long long)empty) - 1;
            empty &= empty - 1;
            if (writer) {
                const float z[VEC] = {};
                const long long row = crd_i ? crd_i[rb + j] : rb + j;
                st_vec<VEC>(A + row * lda + col, z);
            }
        }
    }
    // ---- mode-k coordinate of every leaf of the tile
    for (int q = q0 + tid; q < qend; q += THREADS) {
        int lo = pos_l[q] - t0, hi = pos_l[q + 1] - t0;
        lo = lo < 0 ? 0 : lo;
        hi = hi > cnt ? cnt : hi;
        const int kk = crd_k[q];
        if (hi - lo < LONGF) {
            for (int i = lo; i < hi; ++i) sk[i] = (i == hi - 1) ? ~kk : kk;
        } else {
            const int e = atomicAdd(&nlong, 1);
            if (e < T / LONGF) { slong[3 * e] = kk; slong[3 * e + 1] = lo; slong[3 * e + 2] = hi; }
        }
    }
    __syncthreads();
    {
        const int nl = nlong < T / LONGF ? nlong : T / LONGF;
        for (int e = wave; e < nl; e += NW) {
            const int kk = slong[3 * e], lo = slong[3 * e + 1], hi = slong[3 * e + 2];
            for (int i = lo + lane; i < hi; i += WAVE) sk[i] = (i == hi - 1) ? ~kk : kk;
        }
    }
    __syncthreads();

    // ---- the wave's leaves
    const int CH = T / NW;
    const int wbeg = wave * CH < cnt ? wave * CH : cnt;
    const int wend = wbeg + CH < cnt ? wbeg + CH : cnt;
    float acc[VEC] = {};
    float facc[VEC] = {};                         // sum of b * D(l, :) over the leaves of the open fiber
    bool seen = false;

    auto group_sum = [&](float v) {               // sum over the G lanes that hold the same column
#pragma unroll
        for (int m = GW; m < WAVE; m <<= 1) v += __shfl_xor(v, m, WAVE);
        return v;
    };
    auto flush = [&](int f) {                     // G > 1: acc already holds the sum over the groups
        if (!seen) {
            seen = true;
            if (g == 0) {
#pragma unroll
                for (int v = 0; v < VEC; ++v) srec[2 * wave][gl * VEC + v] = acc[v];
            }
            if (lane == 0) srec_row[2 * wave] = f;
        } else if (writer) {
            const long long row = crd_i ? crd_i[f] : f;
            st_vec<VEC>(A + row * lda + col, acc);
        }
#pragma unroll
        for (int v = 0; v < VEC; ++v) acc[v] = 0.0f;
    };

    // crd_l and vals of 64 leaves, one per lane; requested one batch ahead of their use
    int l_n = 0;
    float v_n = 0.0f;
    auto fetch = [&](int base) {
        l_n = 0;
        v_n = 0.0f;
        if (base + lane < wend) {
            l_n = ld_stream(crd_l + t0 + base + lane);
            v_n = ld_stream(vals + t0 + base + lane);
        }
    };
    fetch(wbeg);
    for (int base = wbeg; base < wend; base += WAVE) {
        const int n = wend - base < WAVE ? wend - base : WAVE;
        const int l_l = l_n;
        const float v_l = v_n;
        int k_l = lane < n ? sk[base + lane] : 0;
        const int f_l = lane < n ? sflag[base + lane] : -1;
        fetch(base + WAVE);
        if (base + lane == wend - 1 && k_l >= 0) k_l = ~k_l;   // the wave's last leaf closes its fiber's partial sum
        if constexpr (G > 1) {
        for (int j0 = 0; j0 < n; j0 += U * G) {
            float c[U], d[U], a[U];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int jj = (j0 + u * G + g) & (WAVE - 1);      // this group's leaf in step u
                const long long ll = __shfl(l_l, jj, WAVE);        // lanes past n hold coordinate 0, value 0, no flag
                const int ke = __shfl(k_l, jj, WAVE);
                a[u] = __shfl(v_l, jj, WAVE);
                c[u] = 0.0f;
                if (ke < 0) c[u] = C[(long long)(~ke) * ldc + lcol];   // this group's leaf closes a fiber
                d[u] = D[ll * ldd + lcol];
            }
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int s0 = j0 + u * G;                          // first leaf of the step
                if (s0 < n) {
                    const float term = (s0 + g < n) ? a[u] * d[u] : 0.0f;
                    bool added = false;
#pragma unroll
                    for (int e = 0; e < G; ++e) {
                        if (rl(k_l, (s0 + e) & (WAVE - 1)) < 0) {   // leaf s0 + e is the last of its fiber
                            if (!added && g <= e) { facc[0] += term; added = true; }
                            const float ce = __shfl(c[u], e * GW + gl, WAVE);   // the C row group e fetched
                            acc[0] = fmaf(ce, facc[0], acc[0]);
                            facc[0] = 0.0f;
                            const int f = rl(f_l, (s0 + e) & (WAVE - 1));
                            if (f >= 0) {                           // ... and of its slice
                                acc[0] = group_sum(acc[0]);
                                flush(f);
                            }
                        }
                    }
                    if (!added) facc[0] += term;
                }
            }
        }
        } else {
        for (int j0 = 0; j0 < n; j0 += U) {
            float c[U][VEC], d[U][VEC];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int j = (j0 + u) & (WAVE - 1);       // lanes past n hold coordinate 0, value 0, no flag
                const int ke = rl(k_l, j);
                const long long ll = rl(l_l, j);
                // The C row is needed once per fiber, where its partial sum closes (uniform over the wave).
                if (ke < 0) {
                    ld_vec<VEC>(c[u], C + (long long)(~ke) * ldc + lcol);
                } else {
#pragma unroll
                    for (int v = 0; v < VEC; ++v) c[u][v] = 0.0f;
                }
                ld_vec<VEC>(d[u], D + ll * ldd + lcol);
            }
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int j = j0 + u;
                if (j < n) {
                    const float a = rl(v_l, j);
#pragma unroll
                    for (int v = 0; v < VEC; ++v) facc[v] = fmaf(a, d[u][v], facc[v]);
                    if (rl(k_l, j) < 0) {
#pragma unroll
                        for (int v = 0; v < VEC; ++v) { acc[v] = fmaf(c[u][v], facc[v], acc[v]); facc[v] = 0.0f; }
                        const int f = rl(f_l, j);
                        if (f >= 0) flush(f);
                    }
                }
            }
        }
        }
    }
    if (wbeg < wend) {
        const int slot = seen ? 2 * wave + 1 : 2 * wave;
        if constexpr (G > 1) acc[0] = group_sum(acc[0]);
        if (g == 0) {
#pragma unroll
            for (int v = 0; v < VEC; ++v) srec[slot][gl * VEC + v] = acc[v];
        }
        if (lane == 0) srec_row[slot] = -1;
    }
    __syncthreads();

    // ---- chain the records (wave 0, group 0)
    if (wave != 0 || g != 0) return;
    float run[VEC] = {};
    auto finalize = [&](int r) {
        if (has_carry && r == r0) {
            if (active) {
#pragma unroll
                for (int v = 0; v < VEC; ++v) carry_val[(long long)t * jdim + col + v] = run[v];
            }
            if (lane == 0 && blockIdx.y == 0) carry_row[t] = r;
        } else if (active) {
            const long long row = crd_i ? crd_i[r] : r;
            st_vec<VEC>(A + row * lda + col, run);
        }
#pragma unroll
        for (int v = 0; v < VEC; ++v) run[v] = 0.0f;
    };
    for (int rec = 0; rec < 2 * NW; ++rec) {
        const int code = srec_row[rec];
        if (code == -2) continue;
#pragma unroll
        for (int v = 0; v < VEC; ++v) run[v] += srec[rec][gl * VEC + v];
        if (code >= 0) finalize(code);
    }
    if (straddle) finalize(r1);
}

// A tile whose slices span more than this many (by the table) leaves the empty ones to workgroups at the end of the launch, as the SpMM
// kernels do (it still walks them, which costs 0.6 us per 256).  Not with several chunks of columns, which share the clearing and lose by workgroups between
// them (7569 slices, j = 59 31.5 -> 34.2 us).  us before / by the tile's workgroup, a slice at a time in k_mttkrp_pos / so: 1 M leaves, a run of
// 1000, j = 64 47 / 60 / 38, 128 70 / 71 / 51;  30 000 325 / 496 / 83, 592 / 508 / 109;  200 000 1897 / 2980 / 426, 3816 / 3037 / 450.
constexpr int kGapSlices = 1024;

// j >= 4: a lane owns four adjacent columns and each group of 64/G lanes walks a run of consecutive leaves of its own, with its own
// open fiber and open slice.  A leaf closes where its fiber ends or its group's run does (marked in the staged leaf itself, so
// nothing is written per leaf of a fiber): there the fiber's sum is multiplied by its C row, which is requested with the D rows.  The
// groups of a wave meet in one segmented sum at the end, two records per wave are chained in position order.  blockIdx.y
// walks chunks of 256/G columns.
// Bound by the L2: a row of D that lies there costs 4.0 ps per 128 bytes on the whole chip; rows from memory come at the fabric's 7.5
// TB/s.  What it replaces (k_mttkrp_groups: a record per group, up to 64 of them chained one after the other; single columns per
// lane for j <= 16) and this kernel, us with all launches: 5.8 M leaves, D of 20 000 rows, j = 6 105 -> 59, 16 125 -> 62, 24 127 -> 82, 64 157 -> 129,
// 96 248 -> 187;  1.4 M leaves, j = 12 64 -> 26, 64 60 -> 48;  0.2 M, j = 64 54 -> 28.
// Sums of leaves: even and odd ones apart, groups and records in fp64 (errors, j = 16 1.49e-7 -> 0.82e-7 of the result, 64 1.69 -> 1.25, 200 2.68 ->
// 1.95).
// SMALL: byte offsets into C and D fit 32 bits.  PLAIN: rows of A are stored through the L2.
template <int G, bool SMALL, bool PLAIN>
__global__ __launch_bounds__(256) void k_mttkrp_runs(int nslices, int nnz, const int *__restrict__ crd_i,
                                                     const int *__restrict__ pos_k, const int *__restrict__ crd_k,
                                                     const int *__restrict__ pos_l, const int *__restrict__ crd_l,
                                                     const float *__restrict__ vals, const float *__restrict__ C, long long ldc,
                                                     const float *__restrict__ D, long long ldd, int jdim,
                                                     float *__restrict__ A, long long lda, const int *__restrict__ tile_slice,
                                                     const int *__restrict__ tile_fiber, int *__restrict__ carry_row,
                                                     float *__restrict__ carry_val, int ntiles, int T)
{
    constexpr int THREADS = 256, NW = THREADS / WAVE, GW = WAVE / G, NG = NW * G, U = 4, LD = 8;
    extern __shared__ int smem[];                 // per leaf: {D offset or l | closes, value}, k where it closes, slice that ends
    int2 *const ent = reinterpret_cast<int2 *>(smem);
    int *const kof = smem + 2 * (T + NG);
    unsigned short *const send = reinterpret_cast<unsigned short *>(kof + T);
    __shared__ double srec[2 * NW][GW][4];
    __shared__ int srec_row[2 * NW];              // -2 unused, -1 open segment, >= 0 slice that ended

    const int tid = threadIdx.x, lane = tid & (WAVE - 1);
    const int wave = __builtin_amdgcn_readfirstlane(tid / WAVE);
    const int filler = (int)blockIdx.x - xcd_grid(ntiles);
    if (filler >= 0) {
        clear_gap_rows<1, kGapSlices>(wave * ((int)gridDim.x - xcd_grid(ntiles)) + filler, nslices, [&](long long r) { return pos_l[pos_k[r]]; },
                                      tile_slice, T, A, jdim, lda, crd_i);
        return;
    }
    const int t = xcd_tile(blockIdx.x, ntiles);
    if (t < 0) return;
    const int t0 = t * T;
    const int cnt = (nnz - t0 < T) ? nnz - t0 : T;
    const int t1 = t0 + cnt;
    const int g = lane / GW, gl = lane % GW;
    const int col0 = (blockIdx.y * GW + gl) * 4;
    const bool active = col0 < jdim;
    const int col = col0 < jdim - 4 ? col0 : jdim - 4;      // the last lane shares columns with its neighbour, same values
    // a run of leaves for each group, an odd number of places apart (the groups' reads hit different banks)
    const int run = (cnt + NG - 1) / NG, step = run | 1;
    const unsigned inv = 0xffffffffu / (unsigned)run + 1;            // i / run = i * inv / 2^32 for i < T
    auto place = [&](int i) { return step == run ? i : i + (int)__umulhi((unsigned)i, inv); };

    int l[LD];
    float v[LD];
    const buf_t lb = buffer_of(crd_l + t0, cnt * 4), vb = buffer_of(vals + t0, cnt * 4);
#pragma unroll
    for (int u = 0; u < LD; ++u) {                // (places behind the tile's end read as 0)
        l[u] = __builtin_amdgcn_raw_buffer_load_b32(lb, tid * 4 + u * THREADS * 4, 0, BUFFER_NT);
        v[u] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(vb, tid * 4 + u * THREADS * 4, 0, BUFFER_NT));
    }
    const int r0 = tile_slice[t], r1 = tile_slice[t + 1];
    const int q0 = tile_fiber[t], q1 = tile_fiber[t + 1];
    const int leaf_r0 = pos_l[pos_k[r0]], leaf_r1 = pos_l[pos_k[r1]];   // first leaf of slices r0, r1
    const bool has_carry = (t > 0) && (leaf_r0 < t0);
    const int rbeg = (t == 0) ? 0 : r0;
    const bool straddle = leaf_r1 != t1;          // slice r1 continues into the next tile
    const int rend = straddle ? r1 + 1 : r1;
    const int qend = (pos_l[q1] != t1) ? q1 + 1 : q1;   // fibers with leaves in this tile: q0 .. qend-1
    const bool near = rend - rbeg < 0xfffe;       // the slices' numbers fit 16 bits
    for (int i = tid; i < T / 2; i += THREADS) reinterpret_cast<int *>(send)[i] = 0;
    if (tid < 2 * NW) srec_row[tid] = -2;
    if (tid == 0 && blockIdx.y == 0 && !has_carry) carry_row[t] = -1;
    auto put = [&](float *to, v4f o) {
        if constexpr (PLAIN) *reinterpret_cast<v4f_u *>(to) = o;
        else __builtin_nontemporal_store((v4f_u)o, reinterpret_cast<v4f_u *>(to));
    };
    auto store = [&](int r, v4f o) { put(A + (long long)(crd_i ? crd_i[r] : r) * lda + col, o); };
#pragma unroll
    for (int u = 0; u < LD; ++u) {
        const int i = tid + u * THREADS;
        if (i < cnt) ent[place(i)] = make_int2(SMALL ? (int)((unsigned)l[u] * (unsigned)ldd * 4u) : l[u], __builtin_bit_cast(int, v[u]));
    }
    __syncthreads();

    // ---- a leaf closes where its fiber ends or its run does, and there needs the fiber's k
    for (int q = q0 + tid; q < qend; q += THREADS) {
        int lo = pos_l[q] - t0, hi = pos_l[q + 1] - t0;
        const int kk = crd_k[q];
        lo = lo < 0 ? 0 : lo;
        hi = hi > cnt ? cnt : hi;
        if (lo >= hi) continue;
        auto close = [&](int i) {
            ent[place(i)].x |= SMALL ? 1 : (int)0x80000000u;
            kof[i] = kk;
        };
        for (int b = (lo / run + 1) * run; b < hi; b += run) close(b - 1);
        close(hi - 1);                            // (a fiber that goes on behind the tile: its run ends here)
    }
    // ---- slice ends, zero rows for slices without leaves
    const long long group_off = (long long)g * lda + col;
    const bool gap = gridDim.y == 1 && r1 - (t == 0 ? 0 : r0) > kGapSlices;            // the empty ones are cleared by the last workgroups of the grid
    for (int rb = rbeg + wave * WAVE; rb < rend; rb += THREADS) {
        const int r = rb + lane;
        const bool valid = r < rend;
        const int ps = valid ? pos_l[pos_k[r]] : 0, pe = valid ? pos_l[pos_k[r + 1]] : 1;
        if (valid && pe > ps) {
            const int e = pe - 1 - t0;
            if (e >= 0 && e < cnt) send[e] = (unsigned short)(near ? r - rbeg + 1 : 0xffff);
        }
        each_empty_row<G>(__ballot(valid && !gap && pe == ps), g, [&](int j) {
            if (active) put(crd_i ? A + (long long)crd_i[rb + j + g] * lda + col : A + (long long)(rb + j) * lda + group_off, v4f{});
        });
    }
    __syncthreads();

    auto slice_at = [&](int i) -> int {           // the slice that ends at leaf i of the tile
        if (near) return rbeg + send[i] - 1;
        int lo = r0, hi = r1;                     // a long run of empty slices: max { r : pos_l[pos_k[r]] <= t0 + i }
        while (lo < hi) {
            const int mid = lo + ((hi - lo + 1) >> 1);
            if (pos_l[pos_k[mid]] <= t0 + i) lo = mid; else hi = mid - 1;
        }
        return lo;
    };
    const char *const Cb = reinterpret_cast<const char *>(C + col), *const Db = reinterpret_cast<const char *>(D + col);
    auto row_of_D = [&](int x) -> v4f_u {
        if constexpr (SMALL) return *reinterpret_cast<const v4f_u *>(Db + ((unsigned)x & ~1u));
        else return *reinterpret_cast<const v4f_u *>(Db + (long long)(x & 0x7fffffff) * ldd * 4);
    };
    auto row_of_C = [&](int k) -> v4f_u {
        if constexpr (SMALL) return *reinterpret_cast<const v4f_u *>(Cb + (unsigned)k * (unsigned)ldc * 4u);
        else return *reinterpret_cast<const v4f_u *>(Cb + (long long)k * ldc * 4);
    };
    auto closes = [&](int x) -> bool { return SMALL ? (x & 1) != 0 : x < 0; };
    const int gi = wave * G + g, j0 = gi * run, len = cnt - j0 < run ? cnt - j0 : run, first = gi * step;
    float even[4] = {}, odd[4] = {};              // sum of b * D(l, :) over the leaves of the open fiber, even and odd ones
    float acc[4] = {}, head[4] = {};              // open slice; the first slice that ended in this run, without what lies before
    int hrow = -1;
    auto walk = [&](int i, auto all) {            // U leaves; all: every group has them
        v4f_u d[U], c[U];
        int2 e[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const bool have = all() || i + u < len;
            e[u] = ent[have ? first + i + u : 0];
            d[u] = row_of_D(e[u].x);
            if (have && closes(e[u].x)) c[u] = row_of_C(kof[j0 + i + u]);
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const bool have = all() || i + u < len;
            float(&to)[4] = u & 1 ? odd : even;
#pragma unroll
            for (int q = 0; q < 4; ++q) to[q] = have ? fmaf(__builtin_bit_cast(float, e[u].y), d[u][q], to[q]) : to[q];
            if (have && closes(e[u].x)) {
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    acc[q] = fmaf(c[u][q], even[q] + odd[q], acc[q]);
                    even[q] = odd[q] = 0.0f;
                }
                if (send[j0 + i + u]) {
                    const int r = slice_at(j0 + i + u);
                    if (hrow < 0) {
                        hrow = r;
#pragma unroll
                        for (int q = 0; q < 4; ++q) head[q] = acc[q];
                    } else if (active) store(r, v4f{acc[0], acc[1], acc[2], acc[3]});
#pragma unroll
                    for (int q = 0; q < 4; ++q) acc[q] = 0.0f;
                }
            }
        }
    };
    int i = 0;
    for (; i + U <= run && (long long)cnt >= (long long)(NG - 1) * run + i + U; i += U) walk(i, [] { return true; });
    for (; i < run; i += U) walk(i, [] { return false; });

    // ---- what the groups before this one leave of its first slice
    {
        double x[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) x[q] = (double)acc[q];
        const unsigned long long has = __ballot(hrow >= 0);
        group_segscan<GW, GW>(x, has, g);
        const int lead = has ? __ffsll((long long)has) - 1 : WAVE, lead_g = lead / GW;      // the first group with an end
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const double p = __shfl_up(x[q], GW & (WAVE - 1), WAVE);
            const double h = (double)head[q] + (g == 0 ? 0.0 : p);
            if (has && g == lead_g) srec[2 * wave][gl][q] = h;
            else head[q] = (float)h;
            if (g == G - 1) srec[2 * wave + (has ? 1 : 0)][gl][q] = x[q];
        }
        if (hrow >= 0 && g != lead_g && active) store(hrow, v4f{head[0], head[1], head[2], head[3]});
        if (has && lane == lead) srec_row[2 * wave] = hrow;
        if (lane == 0 && wave * G * run < cnt) srec_row[2 * wave + (has ? 1 : 0)] = -1;
    }
    __syncthreads();

    // ---- chain the records (wave 0, group 0)
    if (wave != 0 || g != 0) return;
    double sum[4] = {};
    auto finalize = [&](int r) {
        const v4f o = {(float)sum[0], (float)sum[1], (float)sum[2], (float)sum[3]};
        if (has_carry && r == r0) {
            if (active) *reinterpret_cast<v4f_u *>(carry_val + (long long)t * jdim + col) = o;
            if (lane == 0 && blockIdx.y == 0) carry_row[t] = r;
        } else if (active) store(r, o);
#pragma unroll
        for (int q = 0; q < 4; ++q) sum[q] = 0.0;
    };
    for (int rec = 0; rec < 2 * NW; ++rec) {
        const int code = srec_row[rec];
        if (code == -2) continue;
#pragma unroll
        for (int q = 0; q < 4; ++q) sum[q] += srec[rec][gl][q];
        if (code >= 0) finalize(code);
    }
    if (straddle) finalize(r1);
}

bool mttkrp_tile_ok(int32_t tile) { return tile == 256 || tile == 512 || tile == 1024 || tile == 2048; }

hipError_t launch_mttkrp_main(int64_t dim_k, int64_t dim_l, int32_t nslices, int32_t nnz, const int32_t *crd_i, const int32_t *pos_k,
                              const int32_t *crd_k, const int32_t *pos_l, const int32_t *crd_l, const float *vals,
                              const float *C, int64_t ldc, const float *D, int64_t ldd, int32_t j, float *A,
                              int64_t lda, int32_t tile, const Workspace &w, const int32_t *tile_fiber,
                              hipStream_t s)
{
    const int ntiles = (int)(((int64_t)nnz + tile - 1) / tile);
    if (ntiles == 0) return hipSuccess;
    const size_t lds = ((size_t)2 * tile + 3 * (size_t)(tile / 32)) * sizeof(int);
#define PSK_GO(K, GRID)                                                                                         \
    PSK_LAUNCH(K, GRID, dim3(256), lds, s, nslices, nnz, crd_i, pos_k, crd_k, pos_l,                            \
                       crd_l, vals, C, (long long)ldc, D, (long long)ldd, j, A, (long long)lda, w.tile_row,         \
                       tile_fiber, w.carry_row, w.carry_val, ntiles, tile)
    const int nx = xcd_grid(ntiles);
    const int64_t most = 0xffffffffll / 4;
    const bool small = ldd <= most / (dim_l > 0 ? dim_l : 1) && ldc <= most / (dim_k > 0 ? dim_k : 1);
    const uintptr_t al = reinterpret_cast<uintptr_t>(C) | reinterpret_cast<uintptr_t>(D) | reinterpret_cast<uintptr_t>(A);
    int vec = 1;                                  // adjacent columns that a lane of the wide kernel can load at once
    if (j > 64 && j % 2 == 0 && ldc % 2 == 0 && ldd % 2 == 0 && lda % 2 == 0 && (al & 7) == 0) vec = 2;
    if (j > 128 && j % 4 == 0 && ldc % 4 == 0 && ldd % 4 == 0 && lda % 4 == 0 && (al & 15) == 0) vec = 4;
    const bool lines = ldd % 32 == 0 && (reinterpret_cast<uintptr_t>(D) & 127) == 0;      // rows of D begin 128-byte lines
#define PSK_RUNS(G)                                                                                             \
    do {                                                                                                         \
        const size_t lds = ((size_t)2 * (tile + 4 * G) + tile) * 4 + (size_t)tile * 2;                           \
        const int chunks = (j + 256 / G - 1) / (256 / G);                                                        \
        const dim3 grid(nx + (chunks == 1 ? spmm_fillers(nslices, kGapSlices) : 0), chunks);                                                      \
        if (small && plain) PSK_GO((k_mttkrp_runs<G, true, true>), grid);                                        \
        else if (small) PSK_GO((k_mttkrp_runs<G, true, false>), grid);                                           \
        else PSK_GO((k_mttkrp_runs<G, false, false>), grid);                                                     \
    } while (0)
    // Few leaves per slice and rows of A that don't fill 64-byte pieces: their parts reach memory one by one, a slice here and one
    // there.  Through the L2 where A fits the memory-side cache (j = 18, a leaf each, A 63 MB 121 -> 49 us, before this kernel 97;  52, 74 MB 99 -> 45, 67;  160, A 194 MB
    // 182 -> 66, 141; no gain below 32 MB); above that whole rows at once (160, 965 MB: 32 columns 947, whole 384;  96, 2367 MB: whole 1211, 64 columns 1674;  but
    // up to 64 columns still through the L2, 0.91 of the time), or the wide kernel where its lanes own two columns and more (160, 300 MB 0.96).
    const bool few = (j % 16 != 0 || lda % 16 != 0 || (reinterpret_cast<uintptr_t>(A) & 63) != 0) && (int64_t)nnz < 5ll * nslices;
    const double a_mb = (double)nslices * (double)lda * 4 / (1 << 20);
    const bool large = few && a_mb > 256, plain = few && a_mb > 32 && (j <= 64 ? (int64_t)nnz < 3ll * nslices : !large);
    // Columns per group of lanes (us, all launches):
    //   few tiles: narrow chunks, so that the runs are short.  100 tiles, j = 24 16 columns 25, 32 31;  64: 16 29, 32 35, 64 46.  357 tiles, 24: 16 27, 32 31;
    //     48: 16 35, 32 37, 64 48;  64: 16 48, 32 38, 64 49;  128: 32 71, 64 61, 128 74.  666 tiles, 24: 16 42, 32 32;  64: 32 55, 64 49;  128: 64 81, 128 70.
    //     448 tiles, 40: 16 61, 32 47, 64 42.  194 tiles, 100: 16 60, 32 46, 64 43
    //   halves: rows of D that begin 128-byte lines and a D above the L2's size: 32 columns, so that the L2s hold the rows of one
    //     chunk at a time.  D 9.8 MB, 2.9 M leaves, 64: 129 -> 90;  12 MB, 18.6 M, 64: 64 columns 557, 32 425;  24 MB, 46.7 M, 64: 1646, 1416, 128: 49 MB 3530,
    //     2969;  but D 4.9 MB, 5.8 M: 129, 132;
    //     more than 128 columns from 5 MB on (256, 6 MB: 3.2 M 420 -> 335, 7.2 M 1782 -> 1186, both in 64 columns)
    //   more than 128 columns (A would be walked twice): the wide kernel (60 000 slices, 200 columns: 359 against 371 in 256 columns), unless
    //     halves (160: 266 -> 196, 256: 374 -> 296), its lanes cannot own two columns, or tiles are few (100: 200 60 -> 45;  up to 370
    //     tiles and more than 5 leaves per slice (whose parts of A are then not what takes the time): 160, 295 tiles 77 -> 43 in 64 columns, 130, 265 to 360 80 -> 57;  fewer: 343 tiles, 3 per slice 105, 135)
    const bool halves = lines && !large && 4 * dim_l * j > (int64_t(j <= 128 ? 6 : 5) << 20);
    const bool some = j > 128 && vec > 1 && ntiles <= 370 && (int64_t)nnz >= 6ll * nslices;
    if (j >= 4 && (j <= 128 || vec == 1 || halves || ntiles <= 256 || some)) {
        if (j <= 8) PSK_RUNS(32);
        else if (j <= 16 || (ntiles <= 450 && j <= 32) || (ntiles <= 300 && j <= 48) || (ntiles <= (j <= 64 ? 200 : 150) && j <= 128)) PSK_RUNS(16);
        else if (large && j > 64 && (j <= 128 || ntiles <= 256)) PSK_RUNS(2);
        else if (large && j > 128) PSK_RUNS(1);
        else if (some && !halves && ntiles > 256) PSK_RUNS(4);
        else if (ntiles > 200 && ntiles <= 450 && j > 96 && j <= 128) PSK_RUNS(4);
        else if (j <= 32 || halves || ntiles <= 450) PSK_RUNS(8);
        else if (j <= 64) PSK_RUNS(4);
        else if (j <= 128) PSK_RUNS(2);
        else PSK_RUNS(1);
    } else if (j < 4) PSK_GO((k_mttkrp_pos<1, 8>), dim3(nx));
    else if (vec == 2) PSK_GO((k_mttkrp_pos<2, 1>), dim3(nx, (j + 127) / 128));
    else PSK_GO((k_mttkrp_pos<4, 1>), dim3(nx, (j + 255) / 256));
#undef PSK_RUNS
#undef PSK_GO
    return take_launch_status();
}

}  // namespace psk
