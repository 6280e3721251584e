// Position-space SpMM for CSR (BS = 1) and BCSR 4x4 (BS = 4), plus the row-split SpMM baseline.
//
// Schedule (appendix "SPMM on a GPU"): the fused (i,j) loop runs over A's positions, split into
// tiles (workgroups) and wave chunks; the dense column index k is split over the 64 lanes of a
// wave; the loop over a wave's positions is innermost.  Generalised from "k = wave width exactly"
// to any k: a lane owns VEC adjacent columns and blockIdx.y walks column chunks of 64*VEC.
#include "psk_dev.h"
#include "psk_internal.h"

namespace psk {

// One workgroup (4 waves) per tile of T positions (a quarter of its positions per wave, consecutive ones) and per
// column chunk.
//
//  - row ends: sflag[i] = r when position t0+i is the last stored position of row r, else -1
//    (filled from the tile's slice of pos; the tile's metadata lives in LDS).  Empty rows in the
//    tile's write range are zero-filled here.
//  - a wave walks its positions 64 at a time: crd / row-end flags / values are loaded one per lane
//    and broadcast with v_readlane, so the address of the B row is wave-uniform and its load is one
//    contiguous 256*VEC-byte access; U B rows are requested before the first FMA.
//  - a row that ends after at least one earlier row end of the same wave is complete: stored to C.
//    The segment before the first row end of a wave, and the one after the last, go to LDS records;
//    wave 0 chains the records in position order: consecutive open segments belong to the row of the
//    next closed one.  A chain whose row began before the tile becomes the tile's carry record; the
//    open chain at the tile's end is stored by this tile if the row began in it, else carried.
//  - a row's even and odd positions are summed apart (blocks: the products of a block first), so that a wave's share of up to
//    3/8 T positions (row tails of other tiles included) makes no larger error than T/4 in one chain: rows of 300 positive
//    products, k = 128, 127e-9 -> 74e-9 of the sum (93e-9 for shares of T/4); 4 x 4 blocks, 8 per row, 103e-9 -> 69e-9.  The time is
//    the same but for short rows and k > 128 (20 000 rows of 4, k = 200: 31.5 -> 32.2 us).
template <int BS, int VEC, TableUse USE>
__global__ __launch_bounds__(256) void k_spmm_pos(int rows, int nnz, const int *__restrict__ pos,
                                                  const int *__restrict__ crd,
                                                  const float *__restrict__ vals,
                                                  const float *__restrict__ B, int k, long long ldb,
                                                  float *__restrict__ C, long long ldc,
                                                  typename TablePtr<USE != TABLE_READ>::type tile_row,
                                                  int *__restrict__ carry_row,
                                                  float *__restrict__ carry_val, int ntiles, int T, int over,
                                                  int search)
{
    constexpr int THREADS = 256, NW = THREADS / WAVE, KW = WAVE * VEC;
    constexpr int U = BS == 1 ? 8 : (BS == 2 ? 4 : (BS == 4 ? 2 : 1));   // positions whose B rows are in flight together
    extern __shared__ int sflag[];                // T + over ints
    __shared__ float srec[2 * NW][BS][KW];
    __shared__ int srec_row[2 * NW];              // -2 unused, -1 open segment, >= 0 row that ended

    const int t = xcd_tile(blockIdx.x, ntiles);
    if (t < 0) return;
    const int tid = threadIdx.x, lane = tid & (WAVE - 1);
    // BS == 1: tell the compiler that the wave index is uniform (scalar loop control).  With blocks the
    // generated code measured 3 % slower that way, so there it stays a per-lane value.
    const int wave = BS == 1 ? __builtin_amdgcn_readfirstlane(tid / WAVE) : tid / WAVE;
    TileSpan span = tile_span<USE>(rows, pos, t, T, nnz, ntiles, over, tile_row, search);
    if constexpr (BS == 4) {                      // in scalar registers (k = 64: 329.4 -> 327.9 us); the others gain nothing
        span.t0 = __builtin_amdgcn_readfirstlane(span.t0);
        span.cnt = __builtin_amdgcn_readfirstlane(span.cnt);
        span.r0 = __builtin_amdgcn_readfirstlane(span.r0);
        span.r1 = __builtin_amdgcn_readfirstlane(span.r1);
        span.rbeg = __builtin_amdgcn_readfirstlane(span.rbeg);
        span.rend = __builtin_amdgcn_readfirstlane(span.rend);
    }
    const int t0 = span.t0, cnt = span.cnt, r0 = span.r0, r1 = span.r1, rbeg = span.rbeg, rend = span.rend;
    const bool has_carry = span.has_carry, straddle = span.straddle;
    const int col = blockIdx.y * KW + lane * VEC;
    const bool active = col < k;
    const int lcol = active ? col : 0;            // lanes past the last column load column 0 and store nothing

    for (int i = tid; i < cnt; i += THREADS) sflag[i] = -1;
    if (tid < 2 * NW) srec_row[tid] = -2;
    if (tid == 0 && blockIdx.y == 0 && !has_carry) carry_row[t] = -1;
    __syncthreads();

    // ---- row ends of this tile, zero rows
    for (int rb = rbeg + wave * WAVE; rb < rend; rb += THREADS) {
        const int r = rb + lane;
        const bool valid = r < rend;
        const int ps = valid ? pos[r] : 0, pe = valid ? pos[r + 1] : 1;
        if (valid && pe > ps) {
            const int e = pe - 1 - t0;
            if (e >= 0 && e < cnt) sflag[e] = r;
        }
        unsigned long long empty = __ballot(valid && pe == ps);
        if constexpr (BS != 4) {                  // (a row's address a scalar: 0.3 M entries, a run of 100 000 rows, k = 114 1500 -> 831 us, when tiles had
            const int base = __builtin_amdgcn_readfirstlane(rb);   // an order in this kernel 1278;  4 x 4 blocks lose by it: k = 64 325.0 -> 326.9)
            each_empty_row<1>(empty, 0, [&](int j) {
                const float z[VEC] = {};
#pragma unroll
                for (int ii = 0; ii < BS; ++ii)
                    if (active) st_vec<VEC>(C + ((long long)(base + j) * BS + ii) * ldc + col, z);
            });
            empty = 0;
        }
        while (empty) {
            const int j = __ffsll((long long)empty) - 1;
            empty &= empty - 1;
            if (active) {
                const float z[VEC] = {};
#pragma unroll
                for (int ii = 0; ii < BS; ++ii) st_vec<VEC>(C + ((long long)(rb + j) * BS + ii) * ldc + col, z);
            }
        }
    }
    __syncthreads();

    // ---- the wave's positions
    const int CH = (cnt + NW - 1) / NW;
    const int wbeg = wave * CH < cnt ? wave * CH : cnt;
    const int wend = wbeg + CH < cnt ? wbeg + CH : cnt;
    float acc[BS][VEC] = {}, odd[BS == 1 ? VEC : 1] = {};      // the open row (BS == 1: its even and its odd positions)
    bool seen = false;

    auto close = [&]() {                          // acc = the whole of the open row
        if constexpr (BS == 1) {
#pragma unroll
            for (int v = 0; v < VEC; ++v) { acc[0][v] += odd[v]; odd[v] = 0.0f; }
        }
    };
    auto flush = [&](int f) {
        close();
        if (!seen) {
            seen = true;
#pragma unroll
            for (int ii = 0; ii < BS; ++ii)
#pragma unroll
                for (int v = 0; v < VEC; ++v) srec[2 * wave][ii][lane * VEC + v] = acc[ii][v];
            if (lane == 0) srec_row[2 * wave] = f;
        } else if (active) {
#pragma unroll
            for (int ii = 0; ii < BS; ++ii) st_vec<VEC>(C + ((long long)f * BS + ii) * ldc + col, acc[ii]);
        }
#pragma unroll
        for (int ii = 0; ii < BS; ++ii)
#pragma unroll
            for (int v = 0; v < VEC; ++v) acc[ii][v] = 0.0f;
    };

    // crd and vals of 64 positions, one per lane; requested one batch ahead of their use
    int c_n = 0;
    float v_n[BS * BS];
    auto fetch = [&](int base) {
        c_n = 0;
#pragma unroll
        for (int e = 0; e < BS * BS; ++e) v_n[e] = 0.0f;
        if (base + lane < wend) {
            const int p = t0 + base + lane;
            c_n = ld_stream(crd + p);
            if constexpr (BS == 1) v_n[0] = ld_stream(vals + p);
            else {
#pragma unroll
                for (int q = 0; q < BS * BS / 4; ++q) {
                    const v4f v = *reinterpret_cast<const v4f *>(vals + (long long)p * (BS * BS) + q * 4);
                    v_n[4 * q + 0] = v.x; v_n[4 * q + 1] = v.y; v_n[4 * q + 2] = v.z; v_n[4 * q + 3] = v.w;
                }
            }
        }
    };
    constexpr bool AHEAD = BS == 1;               // blocks: 16 more registers per lane would cost occupancy
    if (AHEAD) fetch(wbeg);
    for (int base = wbeg; base < wend; base += WAVE) {
        const int n = wend - base < WAVE ? wend - base : WAVE;
        if (!AHEAD) fetch(base);
        const int c_l = c_n;
        const int f_l = lane < n ? sflag[base + lane] : -1;
        float v_l[BS * BS];
#pragma unroll
        for (int e = 0; e < BS * BS; ++e) v_l[e] = v_n[e];
        if (AHEAD) fetch(base + WAVE);
        for (int j0 = 0; j0 < n; j0 += U) {
            float b[U][BS][VEC];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int j = (j0 + u) & (WAVE - 1);       // lanes past n hold column 0, value 0
                const long long c = rl(c_l, j);
#pragma unroll
                for (int ji = 0; ji < BS; ++ji) {
                    if (BS == 1 || active) ld_vec<VEC>(b[u][ji], B + (c * BS + ji) * ldb + lcol);
                    else {
#pragma unroll
                        for (int v = 0; v < VEC; ++v) b[u][ji][v] = 0.0f;
                    }
                }
            }
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int j = j0 + u;
                if (j < n) {
                    if constexpr (BS == 1) {
                        const float a = rl(v_l[0], j);
#pragma unroll
                        for (int v = 0; v < VEC; ++v) {
                            if (u & 1) odd[v] = fmaf(a, b[u][0][v], odd[v]);
                            else acc[0][v] = fmaf(a, b[u][0][v], acc[0][v]);
                        }
                    } else {
#pragma unroll
                        for (int ii = 0; ii < BS; ++ii) {     // the block's share, then one addition to the row
                            float a[BS], p[VEC];
                            if constexpr (BS != 4) {          // (all broadcasts first: 8 x 8 blocks 314 -> 296 us, 4 x 4 324 -> 326)
#pragma unroll
                                for (int ji = 0; ji < BS; ++ji) a[ji] = rl(v_l[ii * BS + ji], j);
#pragma unroll
                                for (int v = 0; v < VEC; ++v) {
                                    p[v] = a[0] * b[u][0][v];
#pragma unroll
                                    for (int ji = 1; ji < BS; ++ji) p[v] = fmaf(a[ji], b[u][ji][v], p[v]);
                                    acc[ii][v] += p[v];
                                }
                            } else {
#pragma unroll
                                for (int ji = 0; ji < BS; ++ji) {
                                    a[ji] = rl(v_l[ii * BS + ji], j);
#pragma unroll
                                    for (int v = 0; v < VEC; ++v) p[v] = ji == 0 ? a[0] * b[u][0][v] : fmaf(a[ji], b[u][ji][v], p[v]);
                                }
#pragma unroll
                                for (int v = 0; v < VEC; ++v) acc[ii][v] += p[v];
                            }
                        }
                    }
                    const int f = rl(f_l, j);
                    if (f >= 0) flush(f);
                }
            }
        }
    }
    if (wbeg < wend) {
        close();
        const int slot = seen ? 2 * wave + 1 : 2 * wave;
#pragma unroll
        for (int ii = 0; ii < BS; ++ii)
#pragma unroll
            for (int v = 0; v < VEC; ++v) srec[slot][ii][lane * VEC + v] = acc[ii][v];
        if (lane == 0) srec_row[slot] = -1;
    }
    __syncthreads();

    // ---- chain the records (wave 0)
    if (wave != 0) return;
    float run[BS][VEC] = {};
    const long long wcarry = (long long)BS * k;
    auto finalize = [&](int r) {
        if (has_carry && r == r0) {
            if (active) {
#pragma unroll
                for (int ii = 0; ii < BS; ++ii)
#pragma unroll
                    for (int v = 0; v < VEC; ++v) carry_val[(long long)t * wcarry + (long long)ii * k + col + v] = run[ii][v];
            }
            if (lane == 0 && blockIdx.y == 0) carry_row[t] = r;
        } else if (active) {
#pragma unroll
            for (int ii = 0; ii < BS; ++ii) st_vec<VEC>(C + ((long long)r * BS + ii) * ldc + col, run[ii]);
        }
#pragma unroll
        for (int ii = 0; ii < BS; ++ii)
#pragma unroll
            for (int v = 0; v < VEC; ++v) run[ii][v] = 0.0f;
    };
    for (int rec = 0; rec < 2 * NW; ++rec) {
        const int code = srec_row[rec];
        if (code == -2) continue;
#pragma unroll
        for (int ii = 0; ii < BS; ++ii)
#pragma unroll
            for (int v = 0; v < VEC; ++v) run[ii][v] += srec[rec][ii][lane * VEC + v];
        if (code >= 0) finalize(code);
    }
    if (straddle) finalize(r1);
}

bool spmm_csr_tile_ok(int32_t tile) { return tile == 256 || tile == 512 || tile == 1024 || tile == 2048; }
bool bcsr_tile_ok(int32_t tile) { return tile == 64 || tile == 128 || tile == 256 || tile == 512; }

// Widest per-lane vector the operands allow, not wider than needed to cover k with one chunk.
static int pick_vec(const float *B, int32_t k, int64_t ldb, const float *C, int64_t ldc)
{
    const uintptr_t a = reinterpret_cast<uintptr_t>(B) | reinterpret_cast<uintptr_t>(C);
    int vec = 1;
    if (k > 64 && k % 2 == 0 && ldb % 2 == 0 && ldc % 2 == 0 && (a & 7) == 0) vec = 2;
    if (k > 128 && k % 4 == 0 && ldb % 4 == 0 && ldc % 4 == 0 && (a & 15) == 0) vec = 4;
    return vec;
}

template <int BS>
static hipError_t launch_spmm_pos(int32_t rows, int32_t nnz, const int32_t *pos, const int32_t *crd,
                                  const float *vals, const float *B, int32_t k, int64_t ldb, float *C,
                                  int64_t ldc, int32_t tile, int32_t over, const Workspace &w, hipStream_t s, int search)
{
    const int ntiles = (int)(((int64_t)nnz + tile - 1) / tile);
    if (ntiles == 0) return hipSuccess;
    int vec = pick_vec(B, k, ldb, C, ldc);
    if (BS == 8 && vec == 4) vec = 2;             // 8 x 8 blocks: the LDS records of four columns per lane do not fit
    const int kw = WAVE * vec;
    const dim3 grid(xcd_grid(ntiles), (k + kw - 1) / kw);
    const size_t lds = (size_t)(tile + over) * sizeof(int);
    // Reading and searching as instances of their own: 2 x 2 blocks, 400 000 rows of 10, k = 16 315 -> 305 us, 8 x 8, 100 000 of 6, k = 64 301
    // -> 291;  4 x 4, 250 000 of 8, k = 16 276 -> 272 but k = 64 326 -> 332, so not there, and not for single entries (records).
#define PSK_GO(V)                                                                                              \
    do {                                                                                                       \
        if constexpr (BS == 2 || BS == 8) {                                                                    \
            if (search) PSK_GO_(V, TABLE_SEARCH);                                                              \
            else PSK_GO_(V, TABLE_READ);                                                                       \
        } else PSK_GO_(V, TABLE_EITHER);                                                                       \
    } while (0)
#define PSK_GO_(V, S)                                                                                          \
    PSK_LAUNCH((k_spmm_pos<BS, V, S>), grid, dim3(256), lds, s, rows, nnz, pos, crd, vals, B, k,          \
                       (long long)ldb, C, (long long)ldc, w.tile_row, w.carry_row, w.carry_val, ntiles, tile, over, search)
    if (vec == 4) {
        if constexpr (BS < 8) PSK_GO(4);
    } else if (vec == 2) PSK_GO(2);
    else PSK_GO(1);
#undef PSK_GO_
#undef PSK_GO
    return take_launch_status();
}

hipError_t launch_spmm_csr_main(int32_t rows, int32_t cols, int32_t nnz, const int32_t *pos, const int32_t *crd,
                                const float *vals, const float *B, int32_t k, int64_t ldb, float *C,
                                int64_t ldc, int32_t tile, const Workspace &w, hipStream_t s, int search)
{
    // Groups of lanes or the wide kernel (us, 10^6 rows unless stated):
    //   k <= 32: groups; mean row of 1 / 7 / 16 / 300 entries, k = 16: 43 / 94 / 303 against 54 / 99 / 300 for groups of one column
    //     per lane, which they replace; 10^5 rows of 1000 entries, k = 32: 1252 against 1784
    //   k <= 64: groups when the mean row has 8 entries or more (300: k = 40 356 against 423; 4: 189 against 181)
    //   k <= 128: groups where a lane of the wide kernel could not own two columns and would walk A twice (16: k = 99 1223
    //     against 1776; where it can the wide kernel is 1-3 % faster, k = 128 1190 against 1223)
    const bool groups = k <= 32 || (k <= 64 && nnz >= 8ll * rows) ||
                        (k > 64 && k <= kGroupColumns && pick_vec(B, k, ldb, C, ldc) == 1);
    // Tiles in the order of their sweeps over the columns (launch_tile_sweeps) when rows are long.  It pays where B (MB: b_mb) is larger
    // than the L2 and its rows are used by several of the tiles in flight: a row of B is used by one of cols * rows / nnz rows of A.  us in CSR order / ordered,
    // columns sorted in the rows, 40 M entries, 1000 per row, one of 230: k = 32 641 / 412, k = 128 2647 / 1579;  345: 670 / 502, 2694 / 1940;  460: 687 / 554, 2703 / 2212;  690: 722 /
    // 617, 2726 / 2521;  1035: 750 / 661, 2734 / 2717 (alike with 700 and 4000 per row, 100 M entries, k = 16 and 64).  Columns that are not sorted gain nothing: one of 300 677 / 690,
    // 2728 / 2763;  500 732 / 741, k = 64 1415 / 1535, k = 128 1895 / 2006.  So the line is drawn at 384, where those lose no more than 2 % and the others gain a quarter and more.
    // Shares of the columns per tile (span): 0.73 (700 per row, k = 256, 59 MB) 3783 / 3297, 0.93 413 / 420;  B of 6 MB, 1000 per row, k = 16 41 / 47, k = 32 45 / 49.
    const int32_t over = spmm_overhang(rows, nnz, tile);
    const int64_t ntiles = ((int64_t)nnz + tile - 1) / tile;
    const double span = (double)rows * tile / nnz, b_mb = (double)cols * k * 4 / (1 << 20);
    const bool ordered = ntiles >= 4096 && b_mb >= 8 && span <= 0.8 && (double)cols * rows <= 384.0 * nnz;
    // Columns in chunks, where rows of B begin 128-byte lines and the part of B that the tiles in flight gather from (`reach`: all of it,
    // ordered about span of it) does not fit the L2: one chunk after the other, as wide as fits.  A is read once per chunk.  us
    // whole / 64 / 32 columns at a time, 16 M entries, 16 per row: k = 64, B 5 MB 231 / - / 218, 12 MB 417 / - / 291, 24 MB 516 / - / 449, 80 MB 589 / - / 602;
    //   k = 128, 5 MB 414 / 367 / 427, 12 MB 798 / 525 / 429, 40 MB 1082 / 1001 / 842;  k = 256, 12 MB 1600 / 717 / 837, 40 MB 2196 / 1525 / 1038, 80 MB 2320 /
    //   1994 / 1706.  4 per row: k = 64, 24 MB 615 / - / 594, 40 MB 637 / - / 667.  Ordered, 1000 per row: k = 128, 49 MB 1824 / 1632 / 1262, 15 MB 644 / 675 / 763;  k = 64,
    //   24 MB 824 / - / 641, 12 MB 657 / - / 697;  4000 per row, k = 128, 49 MB 790 / 942 / 1048.
    //   Up to which size (whole / 32, 8 M entries): 16 per row, k = 64, 38 MB 282 / 269, 50 MB 293 / 285, 75 MB 299 / 306;  96, 60 MB 414 / 414, 80 MB 421 / 439;  128, 81 MB 577 / 549,
    //   162 MB 593 / 609;  256, 162 MB 1202 / 1090, 216 MB 1207 / 1147, 324 MB 1204 / 1203 (64 per row alike);  4 per row, 64, 24 MB 313 / 303, 28 MB 317 / 315, 38 MB 325 / 337;  128, 59 MB 658 / 637, 81 MB
    //   670 / 674;  96, 44 MB 498 / 490, 60 MB 507 / 513;  256, 119 MB 1396 / 1262, 324 MB 1391 / 1442: 32 columns of 24 MB, 13.5 with few entries per row.
    const bool lines = ldb % 32 == 0 && (reinterpret_cast<uintptr_t>(B) & 127) == 0;
    // Rows of C that fill 64-byte pieces can be stored past the L2 as they come.  Others share a piece with their neighbours, which the kernels
    // with a wave per tile store at other times: with few entries per row that is most of what these kernels do, and then the L2 has to put the
    // pieces together (`plain` stores, while C fits the memory-side cache) or a workgroup stores neighbouring rows at once.
    const bool pieces = spmm_pieces(C, k, ldc);
    const double reach = ordered ? span * b_mb : b_mb, fits = ordered ? 8.2 : 4.2, per = (double)nnz / rows;
    const int vec = pick_vec(B, k, ldb, C, ldc);
    const int32_t whole = k <= 256 ? k : 256;
    int32_t chunk = whole;
    if (lines && reach > fits && k >= 64 && k % 32 == 0) {
        int32_t c = 128;
        while (c > 32 && (c >= k || k % c != 0 || reach * c / k > fits)) c /= 2;
        if (ordered || reach * c / k <= (per >= 8 ? 24.0 : 13.5)) chunk = c;
    }
    // A chunk as large as the part of B that fits gains little where B is a little larger than that, and nothing where a row of C is all there is to do:
    // us workgroups / chunks / wave, whole rows: k = 160, 6 per row, B 4.4 MB 200 / 245 / 183;  k = 224, 10 per row, 4.4 MB 213 / 255 / 190;  160, 1 per row, 5 MB
    // 267 / 294 / -, 1.3 per row, 16 MB 300 / 236 / 303;  rows of C of k + 4: 224, 8 per row, 5 MB 121 / 201 / 114, 1 per row 2.5 times;  128, 100 per row, 8 MB 309 / 206 / 298.
    const bool could = chunk < whole && !ordered;
    if (could && !(pieces ? reach > (k <= 128 || (k % 128 == 0 && per >= 2) ? fits : 6.0) && (per >= 1.15 || b_mb > 6.1) : reach > 7 && per >= 8)) chunk = whole;
    const bool chunked = chunk < whole;
    const int32_t *records = nullptr;
    if (ordered) {
        const hipError_t e = launch_tile_sweeps(rows, cols, nnz, pos, crd, tile, over, reach * (chunk < k ? chunk : k) / k > fits, w, s);
        if (e != hipSuccess) return e;
        records = w.tile_cols;
    }
    // A wave per tile (k_spmm_wave) or a workgroup.  The first is limited by the L2, so it gains where B fits it; rows of B from
    // memory come at the fabric's rate in all kernels, and the workgroups' are a little better at that.  us, 4 M entries unless
    // stated, workgroup / wave:
    //   tiles: 1016, B 2 MB 26 / 32 (4 per row, k = 64), 12.5 / 13.8 (100, k = 32);  1953: 40 / 34, 17.4 / 17.3, k = 128 44 / 30;  3906: 70 / 45, 27.2 / 23.3, 74 / 50;
    //     long rows: k = 8, 100 per row: 1953 15.1 / 17.2, 3906 21.8 / 22.2, 7812 34.9 / 33.0;  k = 12, 1563 16 / 19, 2344 17 / 20;  92 and 400 per row, k = 39
    //     1540 20.4 / 19.2, 1975 22.5 / 20.0, k = 60 21.1 / 19.9, 23.7 / 21.7;  72 columns and more from 4.2 MB, 1563 tiles: 53 / 64;  more than 128 in quads: 1563 up to 50 / 60, 3125 up to 53 / 59, 3907 0.8 to 1.0
    //   B 2 MB: 4 per row k = 32 131 / 56;  16, k = 16 52 / 35;  1000, k = 64 60 / 49;  4, k = 6 61 / 57
    //   B 6 MB: 4 per row k = 32 128 / 67;  16, k = 24 68 / 61;  100, k = 24 56 / 62;  1000, k = 32 45 / 49;  100, k = 96 137 / 101;  16, k = 200 209 / 212
    //   B 8 MB: k = 72, 3 per row 53 / 67, 8 per row 154 / 133
    //   B 16 MB and more: 4 per row k = 16 86 / 79, k = 32 131 / 90, 500 MB 145 / 114;  4, k = 64 176 / 184;  100, k = 32 66 / 72;  10^6 rows of 16, 488 MB, k = 128
    //   1224 / 1250;  more than 256 columns (A is walked again): 4 per row 469 / 484, 16 315 / 289
    //   more than 128 in quads, up to two entries per row: 1 to 10 % lost (k = 256, 1 per row 248 / 272, 2.3 per row 911 / 710)
    const bool shorts = nnz < 32ll * rows, quads = k > 128 && vec == 4 && !chunked && !records;
    const int64_t tiles_for_wave = records || chunked                       ? (k <= 8 && !shorts ? 6000 : 1536)
                                   : k <= 8 && !shorts                      ? 6000
                                   : (quads && k < 240) || (k <= 16 && !shorts) ? 3600
                                   : quads                                  ? 2000
                                   : k <= 64 ? 1536
                                             : (k <= 128 && shorts && b_mb > 4.2 ? 2000 : 1536);
    bool wave = k >= 4 && ntiles >= tiles_for_wave && (k <= 256 || per >= 8) &&
                (records || chunked || b_mb <= 4.5 || (shorts && k <= 64 && b_mb <= 6) || (k > 64 && k <= 128 && b_mb <= (per >= 7 ? 8 : 6.1)) ||
                 (k > 8 && k <= 32 && per < 8) || (k > 128 && could && b_mb <= (vec == 1 ? 10 : 6))) &&
                !(quads && per < (ntiles >= 7000 ? 2.15 : 2.5));
    // Few entries per row of C and no whole pieces: `lo`, the entries per row from which a wave per tile with plain stores is the faster one (it is
    // again below 0.75, where most rows are empty).  us workgroup / wave past the L2 / wave plain, 2 M entries: 1 per row, k = 8, B 1 MB 39 / 87 / 32, 4 MB 41 / 89 / 43;
    //   k = 12, 4 MB 54 / 116 / 53, 16 MB 65 / 119 / 73;  k = 24, 4 MB 83 / 126 / 71, 16 MB 90 / 129 / 93;  k = 100, 1 MB 280 / 300 / 187;  2 per row, k = 8, 4 MB 36 / 49 / 32;
    //   k = 24, 4 MB 75 / 72 / 47;  3 per row, k = 8, 6 MB, 4 M 67 / 86 / 80;  k = 72, 8 MB 53 / 67 / 67;  4 per row, k = 40 35 / 24 / 27;  C of 416 MB, k = 13, 1 per row 195 / 496 / 258
    const bool few = wave && !pieces && !chunked && !records && k <= 128 && per < 3.5;
    const bool fits_mall = (double)rows * ldc * 4 <= 256.0 * (1 << 20);
    bool plain = false;
    if (few && per < 0.75) plain = k <= 64;
    else if (few) {
        const double lo = !fits_mall ? 2.6 : k <= 8 ? (b_mb <= 2.1 ? 1.85 : b_mb <= 4.5 ? 2.6 : 3.5) : k <= 16 ? (b_mb <= 4.5 ? 0 : 2.5) :
                          k <= 32 ? (b_mb <= 8 ? 0 : 1.85) : k <= 64 || b_mb <= 2.1 || (per < 1.85 && (b_mb <= 5.1 || vec == 1)) ? 0 : 3.5;
        wave = per >= lo;
        plain = fits_mall;
    }
    if (wave) return launch_spmm_csr_wave(rows, cols, nnz, pos, crd, vals, B, k, ldb, C, ldc, tile, over, chunk, plain, w, s, records);
    if (groups) return launch_spmm_csr_narrow(rows, cols, nnz, pos, crd, vals, B, k, ldb, C, ldc, tile, over, w, s, search, records);
    return launch_spmm_pos<1>(rows, nnz, pos, crd, vals, B, k, ldb, C, ldc, tile, over, w, s, search);
}

hipError_t launch_spmm_bcsr_main(int32_t bs, int32_t brows, int32_t bcols, int32_t nblocks, const int32_t *pos, const int32_t *crd,
                                 const float *vals, const float *B, int32_t k, int64_t ldb, float *C,
                                 int64_t ldc, int32_t tile, const Workspace &w, hipStream_t s, int search)
{
    const int32_t over = spmm_overhang_blocks(brows, nblocks, tile);
    if (spmm_blocks_by_wave(bs, brows, bcols, nblocks, k, C, ldc, tile))
        return launch_spmm_bcsr_wave(bs, brows, bcols, nblocks, pos, crd, vals, B, k, ldb, C, ldc, tile, over, w, s);
    if (bs == 2) return launch_spmm_pos<2>(brows, nblocks, pos, crd, vals, B, k, ldb, C, ldc, tile, over, w, s, search);
    if (bs == 4) return launch_spmm_pos<4>(brows, nblocks, pos, crd, vals, B, k, ldb, C, ldc, tile, over, w, s, search);
    if (bs == 8) return launch_spmm_pos<8>(brows, nblocks, pos, crd, vals, B, k, ldb, C, ldc, tile, over, w, s, search);
    return hipErrorInvalidValue;
}

// Row-split SpMM baseline: one wave per row, lanes over columns (64 at a time), serial over the
// row's positions.
__global__ __launch_bounds__(256) void k_spmm_wave_per_row(int rows, const int *__restrict__ pos,
                                                           const int *__restrict__ crd,
                                                           const float *__restrict__ vals,
                                                           const float *__restrict__ B, int k, long long ldb,
                                                           float *__restrict__ C, long long ldc)
{
    const int lane = threadIdx.x & (WAVE - 1);
    const int r = blockIdx.x * (256 / WAVE) + threadIdx.x / WAVE;
    if (r >= rows) return;
    const int ps = pos[r], pe = pos[r + 1];
    for (int c0 = 0; c0 < k; c0 += WAVE) {
        const int col = c0 + lane;
        float acc = 0.0f;
        if (col < k)
            for (int p = ps; p < pe; ++p) acc = fmaf(vals[p], B[(long long)crd[p] * ldb + col], acc);
        if (col < k) C[(long long)r * ldc + col] = acc;
    }
}

hipError_t launch_spmm_rowsplit(int32_t rows, const int32_t *pos, const int32_t *crd, const float *vals,
                                const float *B, int32_t k, int64_t ldb, float *C, int64_t ldc, hipStream_t s)
{
    if (rows == 0) return hipSuccess;
    PSK_LAUNCH(k_spmm_wave_per_row, dim3((rows + 3) / 4), dim3(256), 0, s, rows, pos, crd, vals, B, k,
                       (long long)ldb, C, (long long)ldc);
    return take_launch_status();
}

}  // namespace psk
