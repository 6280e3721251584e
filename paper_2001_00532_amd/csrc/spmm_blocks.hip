// SpMM over blocks (BCSR, 2 x 2, 4 x 4, 8 x 8) with a wave per tile.
#include "psk_dev.h"
#include "psk_internal.h"

namespace psk {

// As k_spmm_wave for single entries: up to 64 columns; a lane owns four adjacent ones, each group of 64/G lanes walks a run of blocks of its own
// (BS rows of B and the block's values per step, the values with one address per group), block rows that end inside a run are
// stored by its group, and one segmented sum hands each group what the groups before it leave of its first block row.
// The workgroups' kernel gives a column to each of 64 lanes, most of which idle for narrow operands, and waits at barriers with tiles of
// 64 blocks.  Bound by the L2 (a row of B that lies there 4.0 ps per 128 bytes) and the stream of the blocks: 225 000 rows of 8 blocks
// of 4 x 4, k = 8 244 -> 64 us, k = 32 246 -> 165;  8 x 8, 40 000 of 20, k = 16 349 -> 100;  2 x 2, 40 000 of 20, k = 8 65 -> 23.
// SMALL: byte offsets into B fit 32 bits.  PLAIN: rows of C are stored through the L2.
template <int BS, int G, bool SMALL, bool PLAIN>
__global__ __launch_bounds__(256) void k_spmm_wave_blocks(int rows, int nnz, const int *__restrict__ pos, const int *__restrict__ crd,
                                                          const float *__restrict__ vals, const float *__restrict__ B, int k,
                                                          long long ldb, float *__restrict__ C, long long ldc,
                                                          const int *__restrict__ tile_row, int *__restrict__ carry_row,
                                                          float *__restrict__ carry_val, int ntiles, int T, int over)
{
    constexpr int GW = WAVE / G, U = BS == 2 ? 4 : (BS == 4 ? 2 : 1), GAP = spmm_gap_rows(G, BS);
    typedef v4f_u V;
    extern __shared__ int smem[];
    const int lane = threadIdx.x & (WAVE - 1), g = lane / GW, gl = lane % GW;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / WAVE);
    int *const ent = smem + wave * (T + over);                          // block column, bit 31: a block row ends
    unsigned short *const srow = reinterpret_cast<unsigned short *>(smem + 4 * (T + over)) + wave * (T + over);   // which
    const int quads = (ntiles + 3) / 4, filler = (int)blockIdx.x - xcd_grid(quads);
    if (filler >= 0) {
        clear_gap_rows<BS, GAP>(wave * ((int)gridDim.x - xcd_grid(quads)) + filler, rows, [&](long long r) { return pos[r]; }, tile_row, T, C, k, ldc, nullptr);
        return;
    }
    const int quad = xcd_tile(blockIdx.x, quads), t = quad * 4 + wave;
    if (quad < 0 || t >= ntiles) return;          // (no barriers: waves don't wait for each other)
    const int col0 = gl * 4;
    const bool active = col0 < k;
    const int col = col0 < k - 4 ? col0 : k - 4;

    const TileSpan s = tile_span<TABLE_READ>(rows, pos, t, T, nnz, ntiles, over, tile_row, 0);
    const int t0 = __builtin_amdgcn_readfirstlane(s.t0), cnt = __builtin_amdgcn_readfirstlane(s.cnt);
    const int r0 = __builtin_amdgcn_readfirstlane(s.r0), r1 = __builtin_amdgcn_readfirstlane(s.r1);
    const int rbeg = __builtin_amdgcn_readfirstlane(s.rbeg), rend = __builtin_amdgcn_readfirstlane(s.rend);
    if (lane == 0 && !s.has_carry) carry_row[t] = -1;
    const bool near = rend - rbeg < 0xffff;       // the rows' numbers fit 16 bits
    const bool gap = r1 - (t == 0 ? 0 : r0) > GAP;       // the empty rows are cleared by the last workgroups of the grid

    auto row_at = [&](int i) -> int {             // the block row that ends at position i of the tile
        if (near) return rbeg + srow[i];
        int row[1];
        rows_by_search<1>(pos, r0, r1, {t0 + i}, row);
        return row[0];
    };
    auto put = [&](float *to, V v) {
        if constexpr (PLAIN) *reinterpret_cast<V *>(to) = v;
        else __builtin_nontemporal_store(v, reinterpret_cast<V *>(to));
    };
    auto store = [&](int r, const float (&o)[BS][4]) {
#pragma unroll
        for (int ii = 0; ii < BS; ++ii) put(C + ((long long)r * BS + ii) * ldc + col, V{o[ii][0], o[ii][1], o[ii][2], o[ii][3]});
    };
    auto emit = [&](int r, const float (&o)[BS][4]) {              // a block row that may have begun in an earlier tile
        if (s.has_carry && r == r0) {
#pragma unroll
            for (int ii = 0; ii < BS; ++ii)
                *reinterpret_cast<V *>(carry_val + ((long long)t * BS + ii) * k + col) = V{o[ii][0], o[ii][1], o[ii][2], o[ii][3]};
            if (gl == 0) carry_row[t] = r;
        } else store(r, o);
    };

    for (int i = lane; i < cnt; i += WAVE) ent[i] = ld_stream(crd + t0 + i);
    wave_fence();
    auto mark = [&](int e, int row) {             // position e of the tile ends the block row
        ent[e] |= (int)0x80000000u;
        srow[e] = (unsigned short)(near ? row - rbeg : 0);
    };
    const long long group_off = (long long)g * BS * ldc + col;
    auto row_step = [&](int rb, int from, int to) {                 // block rows rb .. rb + 63, one per lane with its positions
        const bool valid = rb + lane < rend;
        const int e = to - 1 - t0;
        if (valid && to > from && e >= 0 && e < cnt) mark(e, rb + lane);
        each_empty_row<G>(__ballot(valid && to == from), g, [&](int j) {
            float *const at = C + (long long)(rb + j) * BS * ldc + group_off;
#pragma unroll
            for (int ii = 0; ii < BS; ++ii)
                if (active) put(at + ii * ldc, V{});
        });
    };
    if (gap || rend - rbeg <= WAVE) {
        const int q = min(rbeg + lane, rend);     // (pos has an entry behind the last row)
        if (!gap && rend > rbeg) row_step(rbeg, pos[q], pos[min(q + 1, rend)]);
    } else {                                      // (with one step requested at a time each waits for its own)
#pragma unroll 1
        for (int rb = rbeg; rb < rend; rb += 4 * WAVE) {
            int from[4], to[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const int q = min(rb + u * WAVE + lane, rend - 1);
                from[u] = pos[q];
                to[u] = pos[q + 1];
            }
#pragma unroll
            for (int u = 0; u < 4; ++u) row_step(rb + u * WAVE, from[u], to[u]);
        }
    }
    for (int i = lane; gap && i < cnt; i += 2 * WAVE) {
        const int p[2] = {t0 + i, t0 + min(i + WAVE, cnt - 1)};
        int row[2];
        rows_by_search(pos, r0, r1, p, row);
        if (pos[row[0] + 1] == p[0] + 1) mark(i, row[0]);
        if (i + WAVE < cnt && pos[row[1] + 1] == p[1] + 1) mark(i + WAVE, row[1]);
    }
    wave_fence();
    if (cnt <= 0) return;

    const int run = (cnt + G - 1) / G, j0 = g * run, len = cnt - j0 < run ? cnt - j0 : run;
    const float *const tv = vals + (long long)t0 * (BS * BS);
    const char *const Bb = reinterpret_cast<const char *>(B + col);
    constexpr bool TWO = BS == 2;                 // even and odd blocks apart (2 x 2: else the longer chains make larger errors)
    float acc[BS][4] = {}, odd[TWO ? BS : 1][4] = {}, head[BS][4] = {};
    auto join = [&]() {
        if constexpr (TWO) {
#pragma unroll
            for (int ii = 0; ii < BS; ++ii)
#pragma unroll
                for (int q = 0; q < 4; ++q) { acc[ii][q] += odd[ii][q]; odd[ii][q] = 0.0f; }
        }
    };
    int hrow = -1;                                // block row of the first end in this group's run; its sum, without what lies before, in head
    auto walk = [&](int i, auto all) {
        V b[U][BS];
        float a[U][BS * BS];
        int e[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int j = all() || i + u < len ? j0 + i + u : 0;    // (lanes without a block read the tile's first one)
            e[u] = ent[j];
            const int c = e[u] & 0x7fffffff;
#pragma unroll
            for (int ji = 0; ji < BS; ++ji) {
                if constexpr (SMALL) b[u][ji] = *reinterpret_cast<const V *>(Bb + ((unsigned)c * BS + ji) * (unsigned)(ldb * 4));
                else b[u][ji] = *reinterpret_cast<const V *>(Bb + ((long long)c * BS + ji) * ldb * 4);
            }
#pragma unroll
            for (int q = 0; q < BS * BS / 4; ++q) {
                const V v = *reinterpret_cast<const V *>(tv + (unsigned)j * (BS * BS) + q * 4);
#pragma unroll
                for (int x = 0; x < 4; ++x) a[u][4 * q + x] = v[x];
            }
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const bool have = all() || i + u < len;
            if (have) {
#pragma unroll
                for (int ii = 0; ii < BS; ++ii) {                   // the block's share, then one addition to the row
#pragma unroll
                    for (int q = 0; q < 4; ++q) {
                        float p = a[u][ii * BS] * b[u][0][q];
#pragma unroll
                        for (int ji = 1; ji < BS; ++ji) p = fmaf(a[u][ii * BS + ji], b[u][ji][q], p);
                        if constexpr (TWO) { if (u & 1) odd[ii][q] += p; else acc[ii][q] += p; }
                        else acc[ii][q] += p;
                    }
                }
                if (e[u] < 0) {
                    join();
                    const int r = row_at(j0 + i + u);
                    if (hrow < 0) {
                        hrow = r;
#pragma unroll
                        for (int ii = 0; ii < BS; ++ii)
#pragma unroll
                            for (int q = 0; q < 4; ++q) head[ii][q] = acc[ii][q];
                    } else if (active) store(r, acc);
#pragma unroll
                    for (int ii = 0; ii < BS; ++ii)
#pragma unroll
                        for (int q = 0; q < 4; ++q) acc[ii][q] = 0.0f;
                }
            }
        }
    };
    int i = 0;
    for (; i + U <= cnt - (G - 1) * run; i += U) walk(i, [] { return true; });      // (the last group has no more than the others)
    for (; i < run; i += U) walk(i, [] { return false; });

    join();
    // what the groups before this one leave of its first block row: sums of the groups' open ends, afresh after each end
    const unsigned long long has = __ballot(hrow >= 0);
#pragma unroll
    for (int ii = 0; ii < BS; ++ii) {
        group_segscan<GW, GW>(acc[ii], has, g);
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const float p = __shfl_up(acc[ii][q], GW & (WAVE - 1), WAVE);
            head[ii][q] += g == 0 ? 0.0f : p;
        }
    }
    if (hrow >= 0 && active) emit(hrow, head);
    if (s.straddle && g == G - 1 && active) emit(r1, acc);         // the open row goes on in the next tile
}

template <int BS>
static void launch_blocks(int32_t rows, int32_t cols, int32_t nnz, const int32_t *pos, const int32_t *crd, const float *vals, const float *B,
                          int32_t k, int64_t ldb, float *C, int64_t ldc, int32_t tile, int32_t over, const Workspace &w, hipStream_t s)
{
    const int ntiles = (int)(((int64_t)nnz + tile - 1) / tile);
    const bool small = ldb <= 0xffffffffll / 4 / (cols > 0 ? (int64_t)cols * BS : 1);
    const bool plain = small && spmm_blocks_plain(rows, nnz, BS, C, k, ldc);
    const unsigned nx = (unsigned)xcd_grid((ntiles + 3) / 4), fillers = (unsigned)spmm_fillers(rows, spmm_gap_rows(1, BS)), lds = 4u * (unsigned)(tile + over) * 6u;
#define PSK_GO_(GG, SM, PL)                                                                                       \
    PSK_LAUNCH((k_spmm_wave_blocks<BS, GG, SM, PL>), dim3(nx + fillers), dim3(256), lds, s, rows, nnz, pos, crd, \
               vals, B, k, (long long)ldb, C, (long long)ldc, w.tile_row, w.carry_row, w.carry_val, ntiles, tile, over)
#define PSK_GO(GG) do { if (plain) PSK_GO_(GG, true, true); else if (small) PSK_GO_(GG, true, false); else PSK_GO_(GG, false, false); } while (0)
    if (k <= 8) PSK_GO(32);
    else if (k <= 16) PSK_GO(16);
    else if (k <= 32) PSK_GO(8);
    else PSK_GO(4);
#undef PSK_GO
#undef PSK_GO_
}

hipError_t launch_spmm_bcsr_wave(int32_t bs, int32_t brows, int32_t bcols, int32_t nblocks, const int32_t *pos, const int32_t *crd,
                                 const float *vals, const float *B, int32_t k, int64_t ldb, float *C, int64_t ldc, int32_t tile,
                                 int32_t over, const Workspace &w, hipStream_t s)
{
    if (nblocks <= 0) return hipSuccess;
    if (k < 4 || k > 64) return hipErrorInvalidValue;
    if (bs == 2) launch_blocks<2>(brows, bcols, nblocks, pos, crd, vals, B, k, ldb, C, ldc, tile, over, w, s);
    else if (bs == 4) launch_blocks<4>(brows, bcols, nblocks, pos, crd, vals, B, k, ldb, C, ldc, tile, over, w, s);
    else if (bs == 8) launch_blocks<8>(brows, bcols, nblocks, pos, crd, vals, B, k, ldb, C, ldc, tile, over, w, s);
    else return hipErrorInvalidValue;
    return take_launch_status();
}

}  // namespace psk
