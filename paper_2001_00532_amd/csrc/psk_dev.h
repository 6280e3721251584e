// Device-side helpers shared by the kernels (gfx950, wave64).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace psk {

constexpr int WAVE = 64;
constexpr int NUM_XCD = 8;   // MI355X: 8 accelerator dies, workgroups are dealt to them round-robin

typedef int   v4i __attribute__((ext_vector_type(4)));
typedef float v4f __attribute__((ext_vector_type(4)));
typedef float v2f __attribute__((ext_vector_type(2)));

// Streamed-once data (crd, vals): mark the loads non-temporal so they do not push
// the gathered operand out of L2.
template <typename T>
__device__ __forceinline__ T ld_stream(const T *p) { return __builtin_nontemporal_load(p); }

// DPP cross-lane move inside a row of 16 lanes; CTRL is the dpp_ctrl immediate.
template <int CTRL>
__device__ __forceinline__ float dpp_mov(float v)
{
    return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), CTRL, 0xF, 0xF, true));
}

// Sum over the 64 lanes of a wave; every lane receives the same bits.
// Butterfly: quad_perm xor1, quad_perm xor2, row_half_mirror, row_mirror (DPP),
// then xor16 / xor32 through the LDS crossbar.
__device__ __forceinline__ float wave_sum(float v)
{
    v += dpp_mov<0xB1>(v);    // quad_perm [1,0,3,2]
    v += dpp_mov<0x4E>(v);    // quad_perm [2,3,0,1]
    v += dpp_mov<0x141>(v);   // row_half_mirror
    v += dpp_mov<0x140>(v);   // row_mirror
    v += __shfl_xor(v, 16, WAVE);
    v += __shfl_xor(v, 32, WAVE);
    return v;
}

// Tile handled by a workgroup.  Workgroup b runs on die b % 8; give every die one
// contiguous eighth of the tiles so that the part of the dense operand a die
// gathers stays in that die's L2.  Returns -1 for the padding workgroups.
__device__ __forceinline__ int xcd_tile(int bid, int ntiles)
{
    const int per = (ntiles + NUM_XCD - 1) / NUM_XCD;
    const int t = (bid % NUM_XCD) * per + bid / NUM_XCD;
    return (bid / NUM_XCD < per && t < ntiles) ? t : -1;
}
__host__ __device__ __forceinline__ int xcd_grid(int ntiles) { return ((ntiles + NUM_XCD - 1) / NUM_XCD) * NUM_XCD; }

// LDS index skew: one group of `W` words of padding after every 32 words, so that
// per-lane runs whose starts are a multiple of 8/16/32 words apart spread over the banks.
template <int W>
__device__ __forceinline__ int skew(int i) { return i + (i >> 5) * W; }
template <int W>
constexpr int skewed_size(int n) { return n + ((n + 31) >> 5) * W; }

// ---- per-lane vectors of 1, 2 or 4 adjacent dense columns (SpMM, MTTKRP)
template <int VEC> struct VecT;
template <> struct VecT<1> { typedef float type; };
template <> struct VecT<2> { typedef v2f type; };
template <> struct VecT<4> { typedef v4f type; };

template <int VEC>
__device__ __forceinline__ void ld_vec(float (&d)[VEC], const float *p)
{
    typedef typename VecT<VEC>::type V;
    V v = *reinterpret_cast<const V *>(p);
    if constexpr (VEC == 1) d[0] = v;
    else {
#pragma unroll
        for (int i = 0; i < VEC; ++i) d[i] = v[i];
    }
}
template <int VEC>
__device__ __forceinline__ void st_vec(float *p, const float (&s)[VEC])
{
    typedef typename VecT<VEC>::type V;
    V v;
    if constexpr (VEC == 1) v = s[0];
    else {
#pragma unroll
        for (int i = 0; i < VEC; ++i) v[i] = s[i];
    }
    __builtin_nontemporal_store(v, reinterpret_cast<V *>(p));
}

// the same with the alignment of a float only
typedef float v2f_u __attribute__((ext_vector_type(2), aligned(4)));
typedef float v4f_u __attribute__((ext_vector_type(4), aligned(4)));
template <int VEC> struct VecU;
template <> struct VecU<1> { typedef float type; };
template <> struct VecU<2> { typedef v2f_u type; };
template <> struct VecU<4> { typedef v4f_u type; };
template <int VEC>
__device__ __forceinline__ float vec_at(const typename VecU<VEC>::type &v, int i)
{
    if constexpr (VEC == 1) return v;
    else return v[i];
}

// Largest i in [0, n] with a[i] <= target (a non-decreasing, a[0] <= target taken for granted), for two targets at once, by a
// whole wave: every round probes 64 places at equal steps, log64(n) dependent loads instead of log2(n).
__device__ __forceinline__ void wave_search2(const int *__restrict__ a, int n, int target0, int target1, int &r0, int &r1)
{
    const unsigned lane = threadIdx.x & (WAVE - 1);
    unsigned lo0 = 0, hi0 = (unsigned)n, lo1 = 0, hi1 = (unsigned)n;
    while (lo0 < hi0 || lo1 < hi1) {
        const unsigned s0 = (hi0 - lo0 + WAVE - 1) / WAVE, s1 = (hi1 - lo1 + WAVE - 1) / WAVE;
        const unsigned i0 = lo0 + (lane + 1) * s0, i1 = lo1 + (lane + 1) * s1;
        const int v0 = s0 && i0 <= hi0 ? a[i0] : 0x7fffffff, v1 = s1 && i1 <= hi1 ? a[i1] : 0x7fffffff;
        const unsigned c0 = (unsigned)__popcll(__ballot(s0 && i0 <= hi0 && v0 <= target0));
        const unsigned c1 = (unsigned)__popcll(__ballot(s1 && i1 <= hi1 && v1 <= target1));
        lo0 += c0 * s0;
        lo1 += c1 * s1;
        if (s0) hi0 = min(hi0, lo0 + s0 - 1);
        if (s1) hi1 = min(hi1, lo1 + s1 - 1);
    }
    r0 = (int)lo0;
    r1 = (int)lo1;
}

// First row of tile t and of the next one: from the table, or by the kernel's own search, which leaves the table entry for
// the steps that read the table.  (With few tiles the search costs less than the launch of the partition kernel.)
__device__ __forceinline__ void tile_rows(const int *__restrict__ pos, int rows, int nnz, int T, int t, int ntiles, int *tile_row,
                                          int search, int &r0, int &r1)
{
    if (!search) {
        r0 = tile_row[t];
        r1 = tile_row[t + 1];
        return;
    }
    const int c0 = t * T;
    wave_search2(pos, rows, c0, nnz - c0 < T ? nnz : c0 + T, r0, r1);
    if (threadIdx.x == 0 && blockIdx.y == 0) {
        tile_row[t] = r0;
        if (t + 1 == ntiles) tile_row[ntiles] = rows;
    }
}

// The table as a tile kernel sees it: read only (then its loads are scalar), or written by a search.
template <bool SEARCH> struct TablePtr { typedef const int *__restrict__ type; };
template <> struct TablePtr<true> { typedef int *type; };

// What a kernel instance does for its rows: read the table, search, or either by an argument.
enum TableUse { TABLE_READ, TABLE_SEARCH, TABLE_EITHER };

// Positions and rows of tile t where a row that reaches at most `over` positions past the end of a tile is finished by that
// tile (SpMM kernels: a carry record is k floats written, read and added again, a few more positions cost nothing).  A row
// that reaches further ends at the border as the cut says and its part in the next tile becomes that tile's carry.  Both
// tiles at a border decide from pos alone and decide alike; over <= T, so a tile holds at most T + over positions.
struct TileSpan {
    int t0, cnt;           // first position, number of positions (0 when the previous tile took them all)
    int r0, r1;            // table entries
    int rbeg, rend;        // rows written here (rbeg is carried when has_carry)
    bool has_carry;        // row r0 began in an earlier tile
    bool straddle;         // row r1 goes on in the next tile
};
template <TableUse USE = TABLE_EITHER>
__device__ __forceinline__ TileSpan tile_span(int rows, const int *__restrict__ pos, int t, int T, int nnz, int ntiles, int over,
                                              typename TablePtr<USE != TABLE_READ>::type tile_row, int search)
{
    TileSpan s;
    const int c0 = t * T, c1 = nnz - c0 < T ? nnz : c0 + T;
    if constexpr (USE == TABLE_READ) { s.r0 = tile_row[t]; s.r1 = tile_row[t + 1]; }
    else tile_rows(pos, rows, nnz, T, t, ntiles, tile_row, USE == TABLE_SEARCH ? 1 : search, s.r0, s.r1);
    const bool last = t + 1 == ntiles;                    // r1 = rows: no row goes on
    const int b0 = pos[s.r0], e0 = pos[s.r0 + 1], b1 = pos[s.r1], e1 = last ? nnz : pos[s.r1 + 1];
    const bool inside = t > 0 && b0 < c0;                 // the tile begins inside row r0
    const bool taken = inside && e0 - c0 <= over;         // ... whose rest the previous tile took
    s.has_carry = inside && !taken;
    s.rbeg = t == 0 ? 0 : (taken ? s.r0 + 1 : s.r0);
    s.t0 = taken ? e0 : c0;
    const bool open = !last && b1 < c1;                   // row r1 goes on behind the border
    const bool take = open && e1 - c1 <= over;
    s.straddle = open && !take;
    s.rend = open ? s.r1 + 1 : s.r1;
    s.cnt = (take ? e1 : c1) - s.t0;
    return s;
}

// The same as a record of eight ints, so that a tile that is not worked on in CSR order starts with one load instead of the
// chain order -> table -> row positions (which neighbouring workgroups no longer share).
__device__ __forceinline__ void put_record(int *records, long long i, int t, const TileSpan &s)
{
    v4i *p = reinterpret_cast<v4i *>(records + i * 8);
    p[0] = v4i{t, s.t0, s.cnt, s.r0};
    p[1] = v4i{s.r1, s.rbeg, s.rend, (s.has_carry ? 1 : 0) | (s.straddle ? 2 : 0)};
}
__device__ __forceinline__ TileSpan get_record(const int *__restrict__ records, long long i, int &t)
{
    const v4i *p = reinterpret_cast<const v4i *>(records + i * 8);
    const v4i a = p[0], b = p[1];
    TileSpan s;
    t = a.x; s.t0 = a.y; s.cnt = a.z; s.r0 = a.w;
    s.r1 = b.x; s.rbeg = b.y; s.rend = b.z; s.has_carry = b.w & 1; s.straddle = b.w & 2;
    return s;
}

// A range of memory for buffer loads: reads behind `bytes` return 0.
typedef __amdgpu_buffer_rsrc_t buf_t;
constexpr int BUFFER_NT = 2;                      // non-temporal
__device__ __forceinline__ buf_t buffer_of(const void *p, int bytes)
{
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(p), 0, bytes, 0x00020000);
}

// Orders a wave's own reads and writes of LDS.
__device__ __forceinline__ void wave_fence()
{
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

// Sums over the groups of GW lanes of a wave, in fp64: every lane receives the sum of the lanes with its place in a group; and inside
// segments: inclusive sums over groups, a lane of `heads` = its group starts a segment.
template <int GW>
__device__ __forceinline__ double group_sum(double v)
{
#pragma unroll
    for (int d = GW; d < WAVE; d <<= 1) v += __shfl_xor(v, d, WAVE);
    return v;
}
template <int GW, int D, typename T>
__device__ __forceinline__ void group_segscan(T (&x)[4], unsigned long long heads, int g)
{
    if constexpr (D < WAVE) {
        const bool take = g >= D / GW && ((heads >> (threadIdx.x & (WAVE - 1))) & 1) == 0;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const T p = __shfl_up(x[q], D, WAVE);
            x[q] += take ? p : T(0);
        }
        group_segscan<GW, 2 * D>(x, heads | (heads << D), g);
    }
}

// For N positions p[u] of a tile whose table entries are r0 and r1: max { r in [r0, r1] : pos[r] <= p[u] }, the N searches side by side.
template <int N>
__device__ __forceinline__ void rows_by_search(const int *__restrict__ pos, int r0, int r1, const int (&p)[N], int (&row)[N])
{
#pragma unroll
    for (int u = 0; u < N; ++u) row[u] = r0;
    for (unsigned step = r1 > r0 ? 1u << (31 - __builtin_clz(r1 - r0)) : 0; step; step >>= 1) {
#pragma unroll
        for (int u = 0; u < N; ++u) {
            const int at = (int)min((unsigned)row[u] + step, (unsigned)r1);
            row[u] = pos[at] <= p[u] ? at : row[u];
        }
    }
}

// Clears the empty rows (BS rows of C each, k >= 4 columns) of tiles whose rows span more than GAP.  first(r): position at which row r begins;
// tile t owns the rows from its table entry, tile 0 from row 0, to the next entry.  Wave number `index` stands for the rows from index *
// GAP / 4 on (an eighth of a tile's span and less by one wave: a compute unit writes 30 to 40 GB/s, so a span is shared by several; waves that
// follow each other are in different workgroups).  rowmap: the row of C, or nullptr.
template <int BS, int GAP, typename F>
__device__ __forceinline__ void clear_gap_rows(int index, int rows, F first, const int *__restrict__ tile_row, int T,
                                               float *__restrict__ C, int k, long long ldc, const int *__restrict__ rowmap)
{
    constexpr int PART = GAP / 4;
    const long long q = (long long)index * PART;
    if (q >= rows) return;
    const int last = first(q + 1) - 1;            // position before the end of row q: the last tile that owns row q holds it
    const int t = last < 0 ? 0 : last / T;
    const int lo = t == 0 ? 0 : tile_row[t], hi = tile_row[t + 1];
    if (hi - lo <= GAP) return;
    const int beg = q - PART < lo ? lo : (int)q;  // from the tile's first row on where no earlier wave's row lies in it
    const int end = hi - q < PART ? hi : (int)q + PART;
    const int lane = threadIdx.x & (WAVE - 1), quads = (k + 3) / 4;
    int shift = 0;                                // 2^shift lanes per row, `at_once` rows per store
    while (shift < 6 && (1 << shift) < quads) ++shift;
    const int at_once = WAVE >> shift, g = lane >> shift;
    for (long long rb = beg; rb < end; rb += WAVE) {
        const bool mine = rb + lane < end && first(rb + lane) == first(rb + lane + 1);
        const unsigned long long empty = __ballot(mine);
        for (int c = lane & ((1 << shift) - 1); c < quads; c += 1 << shift) {
            const int col = 4 * c < k - 4 ? 4 * c : k - 4;
            float *to = C + (rb + g) * BS * ldc + col;
            for (int i = g; i < WAVE; i += at_once, to += at_once * BS * ldc) {
                if (~empty && !((empty >> i) & 1)) continue;
                float *const at = rowmap ? C + (long long)rowmap[rb + i] * BS * ldc + col : to;
#pragma unroll
                for (int ii = 0; ii < BS; ++ii) *reinterpret_cast<v4f_u *>(at + ii * ldc) = v4f_u{};
            }
        }
    }
}

// Of 64 rows, those of `empty` are cleared, a row by each of the wave's G groups at a time: clear(j) clears row j + g, j the same in all
// lanes (so that a row's address is a scalar and what the lane adds to it, once: with a multiplication per lane each step took 100 ns).
template <int G, typename F>
__device__ __forceinline__ void each_empty_row(unsigned long long empty, int g, F clear)
{
    if (~empty == 0) {
#pragma unroll 4
        for (int j = 0; j < WAVE; j += G) clear(j);
        return;
    }
    while (empty) {
        const int j = __ffsll((long long)empty) - 1;
        if (G == 1 || (j + g < WAVE && ((empty >> ((j + g) & (WAVE - 1))) & 1))) clear(j);
        empty &= ~(((1ull << G) - 1) << j);
    }
}

// ---- per-workgroup trace (only in the instrumented build, -DPSK_CU_TRACE): every workgroup of a traced kernel
// records its start and end on the 100 MHz wall clock and the compute unit it ran on (HW_ID: cu, sh, se;
// XCC_ID: die) into a caller-supplied buffer of 3 x 64 bits per workgroup, from which the host forms each
// CU's busy time.  Each translation unit has its own copy of the pointer; psk_cu_trace_set sets them all.
#ifdef PSK_CU_TRACE
static __device__ unsigned long long *g_cu_trace = nullptr;
static __device__ unsigned g_cu_trace_records = 0;
struct WorkgroupTrace {
    unsigned long long t0;
    __device__ WorkgroupTrace() : t0(wall_clock64()) {}
    __device__ ~WorkgroupTrace()
    {
        if ((threadIdx.x & (WAVE - 1)) == 0 && g_cu_trace && blockIdx.x < g_cu_trace_records) {
            unsigned long long *r = g_cu_trace + 3ull * blockIdx.x;
            atomicMax(r + 1, (unsigned long long)wall_clock64());      // a workgroup ends with its last wave
            if (threadIdx.x == 0) {
                const unsigned hw = __builtin_amdgcn_s_getreg((15 << 11) | (0 << 6) | 4);     // HW_ID[15:0]
                const unsigned xcc = __builtin_amdgcn_s_getreg((3 << 11) | (0 << 6) | 20);    // XCC_ID[3:0]
                r[0] = t0;
                r[2] = (unsigned long long)hw | ((unsigned long long)xcc << 32);
            }
        }
    }
};
inline hipError_t cu_trace_set_here(void *buf, unsigned records)
{
    hipError_t e = hipMemcpyToSymbol(HIP_SYMBOL(g_cu_trace), &buf, sizeof(buf));
    if (e == hipSuccess) e = hipMemcpyToSymbol(HIP_SYMBOL(g_cu_trace_records), &records, sizeof(records));
    return e;
}
#define PSK_TRACE_WORKGROUP() WorkgroupTrace psk_trace_guard_
#else
#define PSK_TRACE_WORKGROUP() do { } while (0)
#endif

// Gathering x for four consecutive positions held by one lane.
//
// The vector-memory address unit takes about one clock per active lane for a gather whatever the
// width of the access (4, 8 or 16 bytes per lane cost the same), so the cheapest gather is the one
// with the fewest lane requests.  Positions whose columns are contiguous (c, c+1, ...: stencils,
// bands, dense blocks) can be served by one 16-byte load of their lane.  run_plan() looks at a lane's
// four columns: run A starts at position 0, run B right after it; if A and B together cover all four
// positions two wide loads replace four narrow ones.  The choice is made per wave (one ballot) so that
// both variants stay straight-line code with every load issued before the first use; unstructured
// matrices never take the wide path and keep their 4-byte gathers.
struct RunPlan { int lenA; int colB; bool ok; };
__device__ __forceinline__ RunPlan run_plan(v4i c, int cols)
{
    const bool e1 = c.y == c.x + 1, e2 = c.z == c.y + 1, e3 = c.w == c.z + 1;
    RunPlan p;
    p.lenA = e1 ? (e2 ? (e3 ? 4 : 3) : 2) : 1;
    p.colB = p.lenA == 1 ? c.y : (p.lenA == 2 ? c.z : c.w);
    const bool covered = p.lenA >= 3 || (p.lenA == 2 && e3) || (p.lenA == 1 && e2 && e3);
    p.ok = covered && c.x <= cols - 4 && p.colB <= cols - 4;
    return p;
}
__device__ __forceinline__ void run_select(const RunPlan &p, v4f_u wA, v4f_u wB, float (&g)[4])
{
    g[0] = wA.x;
    g[1] = p.lenA >= 2 ? wA.y : wB.x;
    g[2] = p.lenA >= 3 ? wA.z : (p.lenA == 2 ? wB.x : wB.y);
    g[3] = p.lenA == 4 ? wA.w : (p.lenA == 3 ? wB.x : (p.lenA == 2 ? wB.y : wB.z));
}

__device__ __forceinline__ int   rl(int v, int lane)   { return __builtin_amdgcn_readlane(v, lane); }
__device__ __forceinline__ float rl(float v, int lane) { return __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, v), lane)); }

}  // namespace psk
