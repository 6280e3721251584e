// CSR SpMM with several positions per step.  The wide SpMM kernel maps the 64 lanes of a wave to 64*VEC columns of B and takes one
// position per step; with few columns most of its instructions are spent on book-keeping per position.  Here a lane owns VEC = 4
// adjacent columns and the wave is split into G groups of 64/G lanes, so that one 16-byte load per lane fetches G rows of B.
//   k_spmm_pos_group: a workgroup per tile, up to 128 columns; the groups take G consecutive positions in one step, every lane keeps the
//     partial sums of its group for the open row, at a row end the sums of the groups are added across the wave.  Row-end flags, records
//     and carries: as in the wide kernel.
//   k_spmm_wave: a wave per tile, any k >= 4 (256/G columns at a time); the groups walk runs of positions of their own.
// The cut is the wide kernel's in both; which of the three takes a product is decided in launch_spmm_csr_main.
#include "psk_dev.h"
#include "psk_internal.h"

namespace psk {

// Sum over the groups of GW lanes: every lane receives the sum of the lanes with its place in a group (rotations inside the
// rows of 16 lanes, then swaps of rows and of halves).
template <int GW>
__device__ __forceinline__ float group_sum(float v)
{
    if (GW <= 1) v += dpp_mov<0x121>(v);    // row_ror:1
    if (GW <= 2) v += dpp_mov<0x122>(v);
    if (GW <= 4) v += dpp_mov<0x124>(v);
    if (GW <= 8) v += dpp_mov<0x128>(v);
    if (GW <= 16) v += __shfl_xor(v, 16, WAVE);
    if (GW <= 32) v += __shfl_xor(v, 32, WAVE);
    return v;
}

// Inclusive sums over groups inside segments of groups; bit g of `heads` = group g starts a segment.
template <int G, int VEC, int D>
__device__ __forceinline__ void group_segscan(float (&v)[VEC], unsigned long long heads, int g)
{
    if constexpr (D < G) {
        constexpr int GW = WAVE / G;
        const bool take = g >= D && ((heads >> g) & 1) == 0;         // no segment starts in groups g-D+1 .. g
#pragma unroll
        for (int i = 0; i < VEC; ++i) {
            const float p = __shfl_up(v[i], GW * D, WAVE);
            v[i] += take ? p : 0.0f;
        }
        group_segscan<G, VEC, 2 * D>(v, heads | (heads << D), g);
    }
}

constexpr int kWaveBlock = 576;                   // positions of a tile that a wave stages at a time

// The last lane of a group whose columns would pass the end of the row takes the last VEC columns instead: it computes and
// stores some of its neighbour's values a second time, bit by bit the same.  So any k >= VEC works, and rows need no
// alignment beyond that of a float.
// SMALL: byte offsets into B fit 32 bits.
template <int G, int VEC, bool SMALL>
__global__ __launch_bounds__(256) void k_spmm_pos_group(int rows, int nnz, const int *__restrict__ pos,
                                                        const int *__restrict__ crd,
                                                        const float *__restrict__ vals,
                                                        const float *__restrict__ B, int k, long long ldb,
                                                        float *__restrict__ C, long long ldc,
                                                        int *tile_row,
                                                        int *__restrict__ carry_row,
                                                        float *__restrict__ carry_val, int ntiles, int T, int over,
                                                  int search, const int *__restrict__ records)
{
    constexpr int THREADS = 256, NW = THREADS / WAVE, GW = WAVE / G, U = G == 32 ? 2 : 4;
    typedef typename VecU<VEC>::type V;
    extern __shared__ int smem[];                 // per position of the tile: {offset or column, value}, row-end flag
    const int TO = T + over;
    int2 *const sent = reinterpret_cast<int2 *>(smem);
    int *const sflag = smem + 2 * TO;
    __shared__ V srec[2 * NW][GW];
    __shared__ int srec_row[2 * NW];              // -2 unused, -1 open segment, >= 0 row that ended

    int t = xcd_tile(blockIdx.x, ntiles);
    if (t < 0) return;
    const int slot = t;
    const int tid = threadIdx.x, lane = tid & (WAVE - 1);
    const int wave = __builtin_amdgcn_readfirstlane(tid / WAVE);
    const int g = lane / GW, gl = lane % GW;
    const bool active = gl * VEC < k;
    const bool writer = active && g == 0;         // group 0 stores on behalf of the wave
    const int col = gl * VEC < k - VEC ? gl * VEC : k - VEC;

    const TileSpan s = records ? get_record(records, slot, t) : tile_span(rows, pos, t, T, nnz, ntiles, over, tile_row, search);
    const int t0 = s.t0, cnt = s.cnt;
    for (int i = tid; i < cnt; i += THREADS) {
        const int c = ld_stream(crd + t0 + i);
        const float v = ld_stream(vals + t0 + i);
        sflag[i] = -1;
        sent[i] = make_int2(SMALL ? (int)((unsigned)c * (unsigned)ldb * 4u) : c, __builtin_bit_cast(int, v));
    }
    if (tid < 2 * NW) srec_row[tid] = -2;
    if (tid == 0 && !s.has_carry) carry_row[t] = -1;
    __syncthreads();

    for (int rb = s.rbeg + wave * WAVE; rb < s.rend; rb += THREADS) {
        const int r = rb + lane;
        const bool valid = r < s.rend;
        const int ps = valid ? pos[r] : 0, pe = valid ? pos[r + 1] : 1;
        if (valid && pe > ps) {
            const int e = pe - 1 - t0;
            if (e >= 0 && e < cnt) sflag[e] = r;
        }
        unsigned long long empty = __ballot(valid && pe == ps);
        while (empty) {
            const int j = __ffsll((long long)empty) - 1;
            empty &= empty - 1;
            if (writer) __builtin_nontemporal_store(V{}, reinterpret_cast<V *>(C + (long long)(rb + j) * ldc + col));
        }
    }
    __syncthreads();

    // the wave's positions: an equal share, rounded up to whole steps
    const int CH = ((cnt + NW - 1) / NW + G - 1) / G * G;
    const int wbeg = wave * CH < cnt ? wave * CH : cnt;
    const int wend = wbeg + CH < cnt ? wbeg + CH : cnt;
    float acc[VEC] = {};                          // this group's share of the open row
    bool seen = false;

    auto group_total = [&](const float (&v)[VEC]) {
        V o;
        if constexpr (VEC == 1) o = group_sum<GW>(v[0]);
        else {
#pragma unroll
            for (int i = 0; i < VEC; ++i) o[i] = group_sum<GW>(v[i]);
        }
        return o;
    };
    const char *const Bb = reinterpret_cast<const char *>(B);
    const unsigned col4 = (unsigned)col * 4u;
    for (int base = wbeg; base < wend; base += WAVE) {
        const int n = wend - base < WAVE ? wend - base : WAVE;
        const int f_l = lane < n ? sflag[base + lane] : -1;
        const unsigned long long ends = __ballot(f_l >= 0);
        for (int j0 = 0; j0 < n; j0 += U * G) {
            V b[U];
            float a[U];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int j = j0 + u * G + g;                       // this group's position in step u
                const int2 e = sent[base + (j < n ? j : 0)];        // behind the end: the value is masked below
                a[u] = __builtin_bit_cast(float, e.y);
                if constexpr (SMALL) b[u] = *reinterpret_cast<const V *>(Bb + ((unsigned)e.x + col4));
                else b[u] = *reinterpret_cast<const V *>(B + (long long)e.x * ldb + col);
            }
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int s0 = j0 + u * G;                          // first position of the step
                if (s0 >= n) break;
                unsigned long long sub = (ends >> s0) & (~0ull >> (64 - G));
                if (sub == 0 && s0 + G <= n) {                      // no row ends here
#pragma unroll
                    for (int v = 0; v < VEC; ++v) acc[v] = fmaf(a[u], vec_at<VEC>(b[u], v), acc[v]);
                } else if (G > 2 && (sub & (sub - 1))) {
                    // two rows or more end here: one segmented sum over the groups serves them all
                    const int first = __ffsll((long long)sub) - 1, last = 63 - __clzll((long long)sub);
                    float term[VEC], x[VEC];
                    const V open = group_total(acc);                // what earlier steps left of the first row
#pragma unroll
                    for (int v = 0; v < VEC; ++v) {
                        term[v] = s0 + g < n ? a[u] * vec_at<VEC>(b[u], v) : 0.0f;
                        x[v] = g == 0 ? term[v] + vec_at<VEC>(open, v) : term[v];
                        acc[v] = g > last ? term[v] : 0.0f;
                    }
                    group_segscan<G, VEC, 1>(x, (sub << 1) | 1, g);
                    V total;
                    if constexpr (VEC == 1) total = x[0];
                    else {
#pragma unroll
                        for (int v = 0; v < VEC; ++v) total[v] = x[v];
                    }
                    const int f = (sub >> g) & 1 ? sflag[base + s0 + g] : -1;
                    if (!seen && g == first) {
                        srec[2 * wave][gl] = total;
                        if (gl == 0) srec_row[2 * wave] = f;
                    } else if (f >= 0 && active) {
                        __builtin_nontemporal_store(total, reinterpret_cast<V *>(C + (long long)f * ldc + col));
                    }
                    seen = true;
                } else {
                    int from = 0;                                   // groups below `from` are done
                    while (sub) {
                        const int e = __ffsll((long long)sub) - 1;
                        sub &= sub - 1;
                        const bool mine = g >= from && g <= e;
#pragma unroll
                        for (int v = 0; v < VEC; ++v)
                            if (mine) acc[v] = fmaf(a[u], vec_at<VEC>(b[u], v), acc[v]);
                        const V total = group_total(acc);
                        const int f = rl(f_l, s0 + e);
                        if (!seen) {
                            seen = true;
                            if (g == 0) srec[2 * wave][gl] = total;
                            if (lane == 0) srec_row[2 * wave] = f;
                        } else if (writer) {
                            __builtin_nontemporal_store(total, reinterpret_cast<V *>(C + (long long)f * ldc + col));
                        }
#pragma unroll
                        for (int v = 0; v < VEC; ++v) acc[v] = 0.0f;
                        from = e + 1;
                    }
                    const bool mine = g >= from && s0 + g < n;
#pragma unroll
                    for (int v = 0; v < VEC; ++v)
                        if (mine) acc[v] = fmaf(a[u], vec_at<VEC>(b[u], v), acc[v]);
                }
            }
        }
    }
    if (wbeg < wend) {
        const V total = group_total(acc);
        const int slot = seen ? 2 * wave + 1 : 2 * wave;
        if (g == 0) srec[slot][gl] = total;
        if (lane == 0) srec_row[slot] = -1;
    }
    __syncthreads();

    // chain the records (wave 0, group 0), in fp64: a tile holds up to 1.5 T positions of a row, and what it took over from the
    // next one no longer meets the rest in the fix-up (rows of 1000 positive products, k = 8: error 39.5e-9 -> 34.2e-9 of the
    // sum, 37.2e-9 without tails; same time)
    if (wave != 0 || g != 0) return;
    double run[VEC] = {};
    auto finalize = [&](int r) {
        V sum;
        if constexpr (VEC == 1) sum = (float)run[0];
        else {
#pragma unroll
            for (int v = 0; v < VEC; ++v) sum[v] = (float)run[v];
        }
        if (s.has_carry && r == s.r0) {
            if (active) *reinterpret_cast<V *>(carry_val + (long long)t * k + col) = sum;
            if (lane == 0) carry_row[t] = r;
        } else if (active) {
            __builtin_nontemporal_store(sum, reinterpret_cast<V *>(C + (long long)r * ldc + col));
        }
#pragma unroll
        for (int v = 0; v < VEC; ++v) run[v] = 0.0;
    };
    for (int rec = 0; rec < 2 * NW; ++rec) {
        const int code = srec_row[rec];
        if (code == -2) continue;
        const V part = srec[rec][gl];
#pragma unroll
        for (int v = 0; v < VEC; ++v) run[v] += (double)vec_at<VEC>(part, v);
        if (code >= 0) finalize(code);
    }
    if (s.straddle) finalize(s.r1);
}

// Many tiles: a wave takes a whole tile, alone, so that no wave waits for another and the chain of dependent loads at a tile's
// start (table, row positions, entries) is paid by a wave among many instead of by a workgroup four times as often.  The tile's
// entries are staged in LDS, up to kWaveBlock at a time, the end of a row marked in the entry itself.
//   no row ends in the tile: the groups take neighbouring positions, every lane adds to its group's share of the open row;
//   else every group walks a run of positions of its own: rows that end inside the run are stored by the group (no sums across
//   lanes), and one segmented sum per block hands each group what the groups before it leave of its first row.
// Bound by the requests to the L2: a row of B in the L2 costs 4.0 ps per 128 bytes on the whole chip however it is asked for, and
// the stream of entries, 8 bytes each from memory, adds 0.8 to 1.7; measured 6.4 ps at k = 32.  Before, us (k_spmm_pos_group / k_spmm_pos, whose
// workgroups wait on barriers) and now: 40 000 rows of 1000 x 25 000, k = 32 360 -> 252;  6000 columns, k = 128 1130 -> 650;  10^6 rows of 16,
// 25 000 columns, k = 16 186 -> 111, k = 32 228 -> 128;  of 5, k = 32 141 -> 75.  Eight steps of loads in flight against four: k = 8 231 -> 205, k = 128
// 705 -> 660; more waves per CU (fewer registers) gain nothing.
template <int G, bool SMALL, bool PLAIN>
__global__ __launch_bounds__(256) void k_spmm_wave(int rows, int nnz, const int *__restrict__ pos, const int *__restrict__ crd,
                                                   const float *__restrict__ vals, const float *__restrict__ B, int k,
                                                   long long ldb, float *__restrict__ C, long long ldc,
                                                   const int *__restrict__ tile_row, int *__restrict__ carry_row,
                                                   float *__restrict__ carry_val, int ntiles, int T, int over,
                                                   const int *__restrict__ records)
{
    constexpr int GW = WAVE / G, U = 8, LD = kWaveBlock / WAVE, GAP = spmm_gap_rows(G, 1);
    constexpr int PLACES = kWaveBlock + G;        // (runs an odd number of places apart)
    typedef v4f_u V;
    extern __shared__ int smem[];
    const int lane = threadIdx.x & (WAVE - 1), g = lane / GW, gl = lane % GW;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / WAVE);
    int2 *const ent = reinterpret_cast<int2 *>(smem) + wave * PLACES;       // {offset or column | row end, value}
    unsigned short *const srow = reinterpret_cast<unsigned short *>(smem + 4 * 2 * PLACES) + wave * kWaveBlock;   // row that ends
    const int quads = (ntiles + 3) / 4, filler = (int)blockIdx.x - xcd_grid(quads);
    if (filler >= 0) {
        if (blockIdx.y == 0) clear_gap_rows<1, GAP>(wave * ((int)gridDim.x - xcd_grid(quads)) + filler, rows, [&](long long r) { return pos[r]; }, tile_row, T, C, k, ldc, nullptr);
        return;
    }
    const int quad = xcd_tile(blockIdx.x, quads), slot = quad * 4 + wave;
    if (quad < 0 || slot >= ntiles) return;                                     // (no barriers: waves don't wait for each other)
    const int col0 = blockIdx.y * (GW * 4) + gl * 4;
    const bool active = col0 < k;
    const int col = col0 < k - 4 ? col0 : k - 4;

    int t = slot;
    TileSpan s = records ? get_record(records, slot, t) : tile_span<TABLE_READ>(rows, pos, t, T, nnz, ntiles, over, tile_row, 0);
    t = __builtin_amdgcn_readfirstlane(t);
    const int t0 = __builtin_amdgcn_readfirstlane(s.t0), cnt = __builtin_amdgcn_readfirstlane(s.cnt);
    const int r0 = __builtin_amdgcn_readfirstlane(s.r0), r1 = __builtin_amdgcn_readfirstlane(s.r1);
    const int rbeg = __builtin_amdgcn_readfirstlane(s.rbeg), rend = __builtin_amdgcn_readfirstlane(s.rend);
    const bool first_y = blockIdx.y == 0;
    const bool gap = r1 - (t == 0 ? 0 : r0) > GAP;       // the empty rows are cleared by the last workgroups of the grid
    const int rwalk = gap ? rbeg : rend;          // rows that are walked

    if (lane == 0 && first_y && !s.has_carry) carry_row[t] = -1;
    // No row ends in this tile, or few do and tiles sweep over the columns together: the groups take neighbouring positions, row by row.
    // (Runs of their own put the groups of a tile at G places of its sweep, all over what the L2 is to hold: 10^5 rows of 1000, k = 32
    // 40.9 M L2 misses and 772 us, so 26.3 M and 690;  40 000 rows, k = 100, B 38 MB 1457 and 1092.  At most 2, 4 or 10 ends: the same.)
    const bool inorder = (s.straddle && rbeg == r1) || (records && rend - rbeg <= 4);
    const bool near = rend - rbeg < 0xffff;       // the rows' numbers fit 16 bits

    const char *const Bb = reinterpret_cast<const char *>(B);
    const unsigned col4 = (unsigned)col * 4u;
    auto row_of_B = [&](int x) -> V {
        if constexpr (SMALL) return *reinterpret_cast<const V *>(Bb + (((unsigned)x & ~1u) + col4));
        else return *reinterpret_cast<const V *>(B + (long long)(x & 0x7fffffff) * ldb + col);
    };
    auto ends_row = [&](int x) -> bool { return SMALL ? (x & 1) != 0 : x < 0; };
    auto row_at = [&](int b0, int i) -> int {     // the row that ends at place i of the block
        if (near) return rbeg + srow[i];
        int row[1];
        rows_by_search<1>(pos, r0, r1, {t0 + b0 + i}, row);
        return row[0];
    };
    auto put = [&](float *to, V v) {
        if constexpr (PLAIN) *reinterpret_cast<V *>(to) = v;
        else __builtin_nontemporal_store(v, reinterpret_cast<V *>(to));
    };
    auto store = [&](int r, const auto (&o)[4]) {
        put(C + (long long)r * ldc + col, V{(float)o[0], (float)o[1], (float)o[2], (float)o[3]});
    };
    auto emit = [&](int r, const double (&o)[4]) {                  // a row that may have begun in an earlier tile
        if (s.has_carry && r == r0) {
            *reinterpret_cast<V *>(carry_val + (long long)t * k + col) = V{(float)o[0], (float)o[1], (float)o[2], (float)o[3]};
            if (gl == 0 && first_y) carry_row[t] = r;
        } else store(r, o);
    };
    auto total = [&](const double (&x)[4], double (&o)[4]) {
#pragma unroll
        for (int q = 0; q < 4; ++q) o[q] = group_sum<GW>(x[q]);
    };

    double open[4] = {};                          // this group's share of the row that is open
    const int nb = (cnt + kWaveBlock - 1) / kWaveBlock, bn = nb ? (cnt + nb - 1) / nb : 0;
    for (int b0 = 0; b0 < cnt || b0 == 0; b0 += bn) {
        const int n = cnt - b0 < bn ? cnt - b0 : bn;
        // a run of positions for each group, an odd number of places apart (the groups' reads hit different banks)
        const int run = (n + G - 1) / G, step = inorder ? run : run | 1;
        const unsigned inv = run > 0 ? 0xffffffffu / (unsigned)run + 1 : 0;               // i / run = i * inv / 2^32 for i < kWaveBlock
        auto place = [&](int i) { return step == run ? i : i + (int)__umulhi((unsigned)i, inv); };
        int pe;                                   // a lane per row: where it ends
        {
            // (places behind the block's end read as 0: the range check of the buffer loads)
            const buf_t cb = buffer_of(crd + t0 + b0, n > 0 ? n * 4 : 0), vb = buffer_of(vals + t0 + b0, n > 0 ? n * 4 : 0);
            int c[LD], r = rbeg + lane;
            float v[LD];
#pragma unroll
            for (int u = 0; u < LD; ++u) {
                c[u] = __builtin_amdgcn_raw_buffer_load_b32(cb, lane * 4 + u * WAVE * 4, 0, BUFFER_NT);
                v[u] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(vb, lane * 4 + u * WAVE * 4, 0, BUFFER_NT));
            }
            int ps = r < rwalk ? pos[r] : 0;
            pe = r < rwalk ? pos[r + 1] : 1;
#pragma unroll
            for (int u = 0; u < LD; ++u) {
                const int i = u * WAVE + lane;
                if (i < n) ent[place(i)] = make_int2(SMALL ? (int)((unsigned)c[u] * (unsigned)ldb * 4u) : c[u], __builtin_bit_cast(int, v[u]));
            }
            wave_fence();
            auto mark = [&](int e, int row) {     // place e of the block ends the row
                ent[place(e)].x |= SMALL ? 1 : (int)0x80000000u;
                srow[e] = (unsigned short)(near ? row - rbeg : 0);
            };
            // (every block of a long tile walks all of the tile's rows: to begin with those of the block costs each tile more, 4 per row, k = 16 44.6 -> 47.0 us)
            const long long group_off = (long long)g * ldc + col;
            auto row_step = [&](int rb, int from, int to) {         // rows rb .. rb + 63, one per lane with its positions
                const int e = to - 1 - t0 - b0;
                if (rb + lane < rwalk && to > from && e >= 0 && e < n) mark(e, rb + lane);
                each_empty_row<G>(b0 == 0 ? __ballot(rb + lane < rwalk && to == from) : 0, g, [&](int j) {
                    if (active) put(C + (long long)(rb + j) * ldc + group_off, V{});
                });
            };
            if (rwalk - rbeg <= 4 * WAVE) {
                for (int rb = rbeg; rb < rwalk; rb += WAVE) {
                    const int from = ps, to = pe;
                    r += WAVE;
                    if (rb + WAVE < rwalk) { ps = r < rwalk ? pos[r] : 0; pe = r < rwalk ? pos[r + 1] : 1; }
                    row_step(rb, from, to);
                }
            } else {                              // (rows of most of them empty: with one step requested ahead each waits for the next)
#pragma unroll 1
                for (int rb = rbeg; rb < rwalk; rb += 4 * WAVE) {
                    int from[4], to[4];
#pragma unroll
                    for (int u = 0; u < 4; ++u) {
                        const int q = min(rb + u * WAVE + lane, rwalk - 1);
                        from[u] = pos[q];
                        to[u] = pos[q + 1];
                    }
#pragma unroll
                    for (int u = 0; u < 4; ++u) row_step(rb + u * WAVE, from[u], to[u]);
                }
            }
            if (gap) {
                constexpr int N = 3;
#pragma unroll 1
                for (int i = lane; i < n; i += N * WAVE) {
                    int p[N], row[N];
#pragma unroll
                    for (int u = 0; u < N; ++u) p[u] = t0 + b0 + min(i + u * WAVE, n - 1);
                    rows_by_search(pos, r0, r1, p, row);
#pragma unroll
                    for (int u = 0; u < N; ++u)
                        if (i + u * WAVE < n && pos[row[u] + 1] == p[u] + 1) mark(i + u * WAVE, row[u]);
                }
            }
            wave_fence();
        }
        if (n <= 0) break;
        if (inorder) {
            auto sweep = [&](int from, int to) {  // positions from .. to - 1 of the block
                for (int i = from; i < to; i += U * G) {
                    V b[U];
                    float a[U], even[4] = {}, odd[4] = {};
#pragma unroll
                    for (int u = 0; u < U; ++u) {
                        const int j = i + u * G + g;
                        const int2 e = ent[j < to ? j : to - 1];
                        a[u] = __builtin_bit_cast(float, e.y);
                        b[u] = row_of_B(e.x);
                    }
                    if (i + U * G <= to) {
#pragma unroll
                        for (int u = 0; u < U; u += 2)
#pragma unroll
                            for (int q = 0; q < 4; ++q) {
                                even[q] = fmaf(a[u], b[u][q], even[q]);
                                odd[q] = fmaf(a[u + 1], b[u + 1][q], odd[q]);
                            }
                    } else {
#pragma unroll
                        for (int u = 0; u < U; ++u)
                            if (i + u * G + g < to) {
                                float(&sum)[4] = u & 1 ? odd : even;
#pragma unroll
                                for (int q = 0; q < 4; ++q) sum[q] = fmaf(a[u], b[u][q], sum[q]);
                            }
                    }
#pragma unroll
                    for (int q = 0; q < 4; ++q) open[q] += (double)(even[q] + odd[q]);
                }
            };
            int at = 0;
            for (int r = rbeg; r < rend; ++r) {
                const int end = __builtin_amdgcn_readlane(pe, r - rbeg) - t0 - b0;
                if (end > n) break;
                // (empty rows, and rows that ended in an earlier block: end <= at; a row whose last position is the first of the tile has end 1)
                if (end <= at) continue;
                sweep(at, end);
                double o[4];
                total(open, o);
                if (active && g == 0) emit(r, o);
#pragma unroll
                for (int q = 0; q < 4; ++q) open[q] = 0.0;
                at = end;
            }
            if (at < n) sweep(at, n);
        } else {
            const int j0 = g * run, len = n - j0 < run ? n - j0 : run;
            const int first = g * step;           // place of the run (lanes without a position read the block's first entry)
            // sums of the open row: the last positions, even and odd ones, and what they were added up to before, as the
            // sum of two floats (a step of Knuth's exact addition: at a row's end cheaper than fp64, 5 per row, k = 32 82 -> 75 us).  Where hi is no longer
            // finite it is the sum, and the step's error (NaN) is left out.  (Here and not at a row's end, which any of the groups may have at any
            // position: 5 per row, k = 32 73.1 us against 75.9, without it 72.6.)
            float even[4] = {}, odd[4] = {}, hi[4] = {}, lo[4] = {}, head[4] = {};
            int hrow = -1;                        // row of the first end in this group's run; its sum, without what lies before, in head
            auto fold = [&]() {
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const float x = even[q] + odd[q], t = hi[q] + x, z = t - hi[q];
                    const float err = (hi[q] - (t - z)) + (x - z);
                    lo[q] += err == err ? err : 0.0f;
                    hi[q] = t;
                    even[q] = odd[q] = 0.0f;
                }
            };
            auto ended = [&](int i) {             // position i of the run ends a row
                const int r = row_at(b0, j0 + i);
                float o[4];
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    o[q] = hi[q] + (lo[q] + (even[q] + odd[q]));
                    even[q] = odd[q] = hi[q] = lo[q] = 0.0f;
                }
                if (hrow < 0) {
                    hrow = r;
#pragma unroll
                    for (int q = 0; q < 4; ++q) head[q] = o[q];
                } else if (active) store(r, o);
            };
            auto walk = [&](int i, auto all) {    // U positions; all: every group has them
                V b[U];
                int2 e[U];
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    e[u] = ent[all() || i + u < len ? first + i + u : 0];
                    b[u] = row_of_B(e[u].x);
                }
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    const bool have = all() || i + u < len;
                    float(&to)[4] = u & 1 ? odd : even;
#pragma unroll
                    for (int q = 0; q < 4; ++q) to[q] = have ? fmaf(__builtin_bit_cast(float, e[u].y), b[u][q], to[q]) : to[q];
                    if (have && ends_row(e[u].x)) ended(i + u);
                }
                fold();
            };
            int i = 0;
            for (; i + U <= n - (G - 1) * run; i += U) walk(i, [] { return true; });      // (the last group has no more than the others)
            for (; i < run; i += U) walk(i, [] { return false; });
            double acc[4];
#pragma unroll
            for (int q = 0; q < 4; ++q) acc[q] = (double)hi[q] + (double)lo[q];
            const unsigned long long has = __ballot(hrow >= 0);
            if (has == 0) {                       // (a tile of several blocks)
#pragma unroll
                for (int q = 0; q < 4; ++q) open[q] += acc[q];
            } else {
                // what the groups before this one leave of its first row: sums of the groups' open ends, afresh after each end
                double before[4], x[4];
                total(open, before);
#pragma unroll
                for (int q = 0; q < 4; ++q) x[q] = g == 0 && hrow < 0 ? acc[q] + before[q] : acc[q];
                group_segscan<GW, GW>(x, has, g);
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const double p = __shfl_up(x[q], GW & (WAVE - 1), WAVE);
                    x[q] = (double)head[q] + (g == 0 ? before[q] : p);
                }
                if (hrow >= 0 && active) emit(hrow, x);
                const int last = 63 - __clzll((long long)has);     // lanes of the last group with an end, and those behind it
#pragma unroll
                for (int q = 0; q < 4; ++q) open[q] = g >= last / GW ? acc[q] : 0.0;
            }
        }
        wave_fence();
    }
    if (s.straddle) {                             // the open row goes on in the next tile
        double o[4];
        total(open, o);
        if (active && g == 0) emit(r1, o);
    }
}

template <int G, int VEC>
static void launch_group(int32_t rows, int32_t nnz, const int32_t *pos, const int32_t *crd, const float *vals, const float *B,
                         int32_t k, int64_t ldb, float *C, int64_t ldc, int32_t tile, int32_t over, bool small,
                         const Workspace &w, hipStream_t s, int search, const int32_t *records)
{
    const int ntiles = (int)(((int64_t)nnz + tile - 1) / tile);
    const dim3 grid(xcd_grid(ntiles));
    const unsigned lds = (unsigned)(tile + over) * 12u;
#define PSK_GO(SM)                                                                                                \
    PSK_LAUNCH((k_spmm_pos_group<G, VEC, SM>), grid, dim3(256), lds, s, rows, nnz, pos, crd, vals, B, k,          \
                       (long long)ldb, C, (long long)ldc, w.tile_row, w.carry_row, w.carry_val, ntiles, tile, over, search, records)
    if (small) PSK_GO(true);
    else PSK_GO(false);
#undef PSK_GO
}

// cols * ldb decides whether 32-bit byte offsets into B are enough
hipError_t launch_spmm_csr_narrow(int32_t rows, int32_t cols, int32_t nnz, const int32_t *pos, const int32_t *crd,
                                  const float *vals, const float *B, int32_t k, int64_t ldb, float *C, int64_t ldc,
                                  int32_t tile, int32_t over, const Workspace &w, hipStream_t s, int search, const int32_t *records)
{
    if (nnz <= 0) return hipSuccess;
    const bool small = ldb <= 0xffffffffll / 4 / (cols > 0 ? cols : 1);
#define PSK_GO(GG, VV) launch_group<GG, VV>(rows, nnz, pos, crd, vals, B, k, ldb, C, ldc, tile, over, small, w, s, search, records)
    if (k < 4) PSK_GO(16, 1);
    else if (k <= 8) PSK_GO(32, 4);
    else if (k <= 16) PSK_GO(16, 4);
    else if (k <= 32) PSK_GO(8, 4);
    else if (k <= 64) PSK_GO(4, 4);
    else if (k <= 128) PSK_GO(2, 4);
    else return hipErrorInvalidValue;
#undef PSK_GO
    return take_launch_status();
}

hipError_t launch_spmm_csr_wave(int32_t rows, int32_t cols, int32_t nnz, const int32_t *pos, const int32_t *crd,
                                const float *vals, const float *B, int32_t k, int64_t ldb, float *C, int64_t ldc,
                                int32_t tile, int32_t over, int32_t chunk, bool plain, const Workspace &w, hipStream_t s, const int32_t *records)
{
    if (nnz <= 0) return hipSuccess;
    if (k < 4) return hipErrorInvalidValue;
    const int ntiles = (int)(((int64_t)nnz + tile - 1) / tile);
    const unsigned nx = (unsigned)xcd_grid((ntiles + 3) / 4);
    const bool small = ldb <= 0xffffffffll / 4 / (cols > 0 ? cols : 1);
    plain = plain && small;
#define PSK_GO_(GG, SM, PL)                                                                                       \
    PSK_LAUNCH((k_spmm_wave<GG, SM, PL>), dim3(nx + (unsigned)spmm_fillers(rows, spmm_gap_rows(GG, 1)), (unsigned)((k + 256 / GG - 1) / (256 / GG))), dim3(256), 4u * ((kWaveBlock + GG) * 8u + kWaveBlock * 2u), s, rows, nnz, pos, crd, vals, B, k, (long long)ldb, C, \
               (long long)ldc, w.tile_row, w.carry_row, w.carry_val, ntiles, tile, over, records)
#define PSK_GO(GG) do { if (plain) PSK_GO_(GG, true, true); else if (small) PSK_GO_(GG, true, false); else PSK_GO_(GG, false, false); } while (0)
    if (chunk <= 8) PSK_GO(32);
    else if (chunk <= 16) PSK_GO(16);
    else if (chunk <= 32) PSK_GO(8);
    else if (chunk <= 64) PSK_GO(4);
    else if (chunk <= 128) PSK_GO(2);
    else PSK_GO(1);
#undef PSK_GO
#undef PSK_GO_
    return take_launch_status();
}

}  // namespace psk
