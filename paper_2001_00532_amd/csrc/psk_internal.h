// Host-side declarations shared between the C-ABI layer (api.hip) and the kernel files.
#pragma once
#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>
#include <tuple>
#include <utility>

namespace psk {

// Kernel launches go through hipLaunchKernel so that each launcher reports the status of ITS launches only:
// the global "last error" of the runtime may hold (and reading it would clear) an error left by the caller's
// own earlier HIP calls.  A launcher may launch several kernels; the first failure is kept per host thread
// and handed out (and reset) by take_launch_status().
extern thread_local hipError_t tls_launch_status;
inline hipError_t take_launch_status()
{
    const hipError_t e = tls_launch_status;
    tls_launch_status = hipSuccess;
    return e;
}
template <typename... KA, size_t... I>
inline hipError_t launch_tuple(void (*kern)(KA...), dim3 grid, dim3 block, unsigned shmem, hipStream_t s,
                               std::tuple<KA...> &args, std::index_sequence<I...>)
{
    void *ptrs[sizeof...(KA) ? sizeof...(KA) : 1] = {static_cast<void *>(&std::get<I>(args))...};
    return hipLaunchKernel(reinterpret_cast<const void *>(kern), grid, block, ptrs, shmem, s);
}
template <typename... KA, typename... A>
inline void launch_kernel(void (*kern)(KA...), dim3 grid, dim3 block, unsigned shmem, hipStream_t s, A &&...a)
{
    static_assert(sizeof...(KA) == sizeof...(A), "argument count does not match the kernel's parameters");
    std::tuple<KA...> args{static_cast<KA>(a)...};
    const hipError_t e = launch_tuple(kern, grid, block, shmem, s, args, std::index_sequence_for<KA...>{});
    if (e != hipSuccess && tls_launch_status == hipSuccess) tls_launch_status = e;
}
#define PSK_LAUNCH(kern, grid, block, shmem, stream, ...) \
    ::psk::launch_kernel(kern, grid, block, shmem, stream, __VA_ARGS__)

// Workspace carving: [tile_row: ntiles+1 int32][carry_row: ntiles int32][carry_val: ntiles*width float]
// [tile_aux: ntiles+1 int32 (second table of a two-level cut)][tile_cols: ntiles*8 int32 (column range of each
// tile, one min/max pair per wave, written by the first column pass)], each part starting on a 256-byte boundary.
struct Workspace {
    int32_t *tile_row;
    int32_t *carry_row;
    float   *carry_val;
    int32_t *tile_aux;
    int32_t *tile_cols;
    size_t   bytes;
};
inline size_t align256(size_t n) { return (n + 255) & ~size_t(255); }
inline Workspace carve(void *base, int64_t ntiles, int64_t width)
{
    Workspace w;
    char *p = static_cast<char *>(base);
    size_t a = align256(size_t(ntiles + 1) * 4), b = align256(size_t(ntiles) * 4 + 4),
           c = align256(size_t(ntiles) * size_t(width) * 4 + 4);
    w.tile_row = reinterpret_cast<int32_t *>(p);
    w.carry_row = reinterpret_cast<int32_t *>(p + a);
    w.carry_val = reinterpret_cast<float *>(p + a + b);
    const size_t d = align256(size_t(ntiles) * 32 + 4);
    w.tile_aux = reinterpret_cast<int32_t *>(p + a + b + c);
    w.tile_cols = reinterpret_cast<int32_t *>(p + a + b + c + a);
    w.bytes = a + b + c + a + d;
    return w;
}

// Every launcher enqueues on `s` and returns the status of its own launches (take_launch_status()).

hipError_t launch_partition(int64_t rows, int64_t nnz, const int32_t *pos, int32_t tile, int method,
                            int32_t *tile_row, hipStream_t s);
hipError_t launch_fill_zero(float *p, int64_t n, hipStream_t s);
// y[crd_i[s]] = sums[s], all other elements 0 (DCSR: row sums in the order of the stored rows)
hipError_t launch_expand_rows(int64_t rows, int32_t nstored, const int32_t *crd_i, const float *sums, float *y, hipStream_t s);
hipError_t launch_fill_zero_2d(float *p, int64_t rows, int32_t width, int64_t ld, hipStream_t s);
hipError_t launch_validate_csr(int32_t rows, int32_t cols, int32_t nnz, const int32_t *pos, const int32_t *crd,
                               int32_t *result, hipStream_t s);
hipError_t launch_max_row(int32_t rows, const int32_t *pos, int32_t *result, hipStream_t s);
hipError_t launch_probe_locality(int32_t nnz, const int32_t *crd, int32_t *result, hipStream_t s);
// Adds the per-tile carry records to the output: element e of a record of `nsub*k` floats goes to
// out[(row*nsub + e / k) * ld + e % k].
// `pos2` (optional): two-level hierarchy, a row's last position is pos2[pos[r+1]] - 1.  `rowmap` (optional):
// row r of the hierarchy is stored at output row rowmap[r].
// over: the tiles take up to that many positions of a row past their end, such a tail has no record (SpMM)
// gap_rows = rows (CSR SpMV only): extra workgroups clear the long runs of empty rows that the tile kernels leave out
hipError_t launch_carry_fixup(int32_t ntiles, int32_t nsub, int32_t k, int64_t ld, int32_t tile, const int32_t *pos,
                              const Workspace &w, float *out, hipStream_t s, const int32_t *pos2 = nullptr,
                              const int32_t *rowmap = nullptr, int32_t gap_rows = 0, int32_t over = 0);
// A tile whose rows span more than this many rows (by the table) does not walk them: it finds the rows of its positions by
// search and leaves the empty rows to the fix-up step.  A workgroup of that step stands for kGapStep rows, looks up the tile
// that owns the first of them and clears its share of the span if the tile is such a one.
constexpr int32_t kGapRows = 32768;
constexpr int32_t kGapStep = 8192;
// Up to this many tiles the tile kernel searches its rows itself and the partition kernel is not launched: 196 tiles 17.4
// -> 14.4 us per product, 1953 tiles 33.4 against 33.2, 3907 tiles (4x4 blocks) 43 -> 48: from a few tiles per CU on the
// searches of the workgroups queue behind each other.
constexpr int32_t kSearchTiles = 1024;

// CSR SpMV
bool spmv_csr_tile_ok(int32_t tile);
hipError_t launch_spmv_csr_main(int32_t rows, int32_t cols, int32_t nnz, const int32_t *pos, const int32_t *crd,
                                const float *vals, const float *x, float *y, int32_t tile, int32_t col_passes,
                                const Workspace &w, hipStream_t s, int search, const int32_t *rowmap = nullptr,
                                bool gaps = false);
// Small matrices: blocks of whole rows, one launch, no table, no carries.  What costs is a long row, which one workgroup sums:
// tiles and fix-up take 10 us whatever the rows are, blocks 7 with 8192 entries in a row, and in one row of scattered columns
// 14.5 with 24 576, 18.6 with 32 768, 27 with 49 152 (fp64 11 with 12 288, 18.4 with 24 576; two rows of half that each 14.7, 11.1).
// So a single row goes by tiles above half the limit.  A row with most of the entries among others is not seen from here.
constexpr int32_t kSmallNnz = 49152, kSmallNnzF64 = 24576, kSmallRows = 65536;
inline bool spmv_small(int64_t rows, int64_t nnz, int vbytes)
{
    const int32_t most = vbytes == 8 ? kSmallNnzF64 : kSmallNnz;
    return nnz > 0 && nnz <= (rows == 1 ? most / 2 : most) && rows <= kSmallRows;
}
// Up to this many entries (fp32) the workspace is not touched and only the main phase does anything.  Above, a phase may be
// followed by one of a call that gives the tile's size or of another entry point with the same table, so what those read is
// there: the partition phase writes the table, the main phase the table and empty carry records (a few dozen words).
constexpr int32_t kNoTableNnz = 16384;
// w (optional): also write the table and empty carry records of tiles of `tile` positions there
hipError_t launch_spmv_csr_small(int32_t rows, int32_t nnz, const int32_t *pos, const int32_t *crd, const float *vals,
                                 const float *x, float *y, int32_t tile, const Workspace *w, hipStream_t s);
hipError_t launch_spmv_csr_small(int32_t rows, int32_t nnz, const int32_t *pos, const int32_t *crd, const double *vals,
                                 const double *x, double *y, int32_t tile, const Workspace *w, hipStream_t s);
// rowmap (optional, both launchers): row r of the hierarchy is row rowmap[r] of y (DCSR)
hipError_t launch_spmv_rowsplit(int32_t rows, const int32_t *pos, const int32_t *crd, const float *vals,
                                const float *x, float *y, int variant, hipStream_t s,
                                const int32_t *rowmap = nullptr);

// CSR SpMV with the position space divided into `parts` pieces of chunks_per_part * 2048 positions
// (persistent workgroups, in-kernel search, no table); carry records: one per part
constexpr int32_t kDivideChunk = 2048;
hipError_t launch_spmv_csr_divide(int32_t rows, int32_t cols, int32_t nnz, const int32_t *pos, const int32_t *crd,
                                  const float *vals, const float *x, float *y, int32_t parts,
                                  int32_t chunks_per_part, const Workspace &w, hipStream_t s);

// CSR SpMV, fp64 operands (carry records are doubles: the workspace is carved with width 2)
bool spmv_csr_f64_tile_ok(int32_t tile);
hipError_t launch_spmv_csr_f64_main(int32_t rows, int32_t cols, int32_t nnz, const int32_t *pos, const int32_t *crd,
                                    const double *vals, const double *x, double *y, int32_t tile, int32_t col_passes,
                                    const Workspace &w, hipStream_t s, int search);
hipError_t launch_carry_fixup_f64(int32_t ntiles, int32_t tile, const int32_t *pos, const Workspace &w, double *out,
                                  hipStream_t s, int32_t gap_rows);

// CSR SpMM
// records of the tiles in w.tile_cols, in the order in which they sweep over the columns (reads the table)
hipError_t launch_tile_sweeps(int32_t rows, int32_t cols, int32_t nnz, const int32_t *pos, const int32_t *crd, int32_t tile,
                              int32_t over, bool tight, const Workspace &w, hipStream_t s);
// The kernels with a wave per tile (k >= 4) neither walk nor clear a long run of empty rows alone: where a tile's rows, by the table, span more than
// `gap`, the wave finds the rows of its positions by search, and workgroups of their own at the end of the same launch clear the empty
// rows.  A wave of theirs stands for `gap` / 4 rows, looks up the tile that owns the first of them and clears what is empty from there to
// the next wave's row if the tile is of this kind (so the row of such a wave lies in every such tile).  us by one wave / so / by the four waves of
// a workgroup per tile (k_spmm_pos_group, k_spmm_pos): one run in 1.9 M entries, k = 64, of 30 000 rows 3403 / 30 / 495, 10^6 115 900 / 76 / 14 600.
// At the head of the launch these workgroups unbalance the tiles: 1.3 M entries in 2 M rows, k = 256 425 -> 472.
// Shorter runs are cleared by the tile's wave, a row to each of its G groups of lanes; a compute unit writes 30 to 40 GB/s, so that costs the
// more the wider the rows are.  us by a workgroup / walked / left to others, 1.5 M entries, 400 per row, a run of 500 | 1000 | 2000: k = 30 31 / 26 / - | 38 / 31 /
// - | 54 / 38 / 28;  64 35 / 31 / - | 43 / 38 / - | 59 / 48 / 31;  100 67 / 52 / 42 | 74 / 62 / 43 | 87 / - / 44;  256 76 / 94 / 68 | 84 / 113 / 70;  4 x 4 blocks, k = 45 34 / 28 / - | 44 / 38 /
// 18 | 64 / - / 19.  Scattered entries, one row in 2.5 (tiles of 1280 rows), where the search is paid by every tile: k = 8 98 / 33 / 40, 48 153 / 129 / 115, 128 274 / 292 / 258.
constexpr int32_t spmm_gap_rows(int groups, int bs) { return bs > 1 ? 512 : (groups <= 2 ? 256 : 1024); }
inline int32_t spmm_fillers(int32_t rows, int32_t gap)        // these workgroups: a multiple of the dies, so that the next chunk of columns meets the same ones
{
    return rows > gap ? (int32_t)(((int64_t)rows + 8 * gap - 1) / (8 * gap)) * 8 : 0;
}
// A row that reaches at most this far past the end of a tile is finished by that tile (tile_span in psk_dev.h).  It saves most of
// the carries when rows are shorter than tiles; CSR rows of half a tile and more would only make the tiles unequal (0.5 to 1.5 T
// positions) and leave few carries less: us with tile / 2 | with 0, tile 512: rows of 30, k = 128 41 | 43;  60 404 | 407;  200 457 | 465 (k = 32
// 87 | 84);  430 162 | 150;  1000 82 | 76, k = 32 in column order 1200 | 875.  Blocks (tile 64) from two tiles on: 4 x 4, k = 128: 8 per
// row 650 | 650;  40 226 | 252;  200 209 | 208;  2 x 2, 300 per row: 142 | 140.
inline int32_t spmm_overhang(int64_t rows, int64_t nnz, int32_t tile) { return 2 * nnz >= rows * tile ? 0 : tile / 2; }
inline int32_t spmm_overhang_blocks(int64_t brows, int64_t nblocks, int32_t tile) { return nblocks >= 2 * brows * tile ? 0 : tile / 2; }
bool spmm_csr_tile_ok(int32_t tile);
hipError_t launch_spmm_csr_main(int32_t rows, int32_t cols, int32_t nnz, const int32_t *pos, const int32_t *crd,
                                const float *vals, const float *B, int32_t k, int64_t ldb, float *C,
                                int64_t ldc, int32_t tile, const Workspace &w, hipStream_t s, int search);
// k <= kGroupColumns: the wave is split into groups that take consecutive positions
constexpr int32_t kGroupColumns = 128;
hipError_t launch_spmm_csr_narrow(int32_t rows, int32_t cols, int32_t nnz, const int32_t *pos, const int32_t *crd,
                                  const float *vals, const float *B, int32_t k, int64_t ldb, float *C, int64_t ldc,
                                  int32_t tile, int32_t over, const Workspace &w, hipStream_t s, int search, const int32_t *records);
// k >= 4, many tiles: a wave per tile (reads the table) and per `chunk` columns, up to 256; plain: rows of C are stored through the L2
hipError_t launch_spmm_csr_wave(int32_t rows, int32_t cols, int32_t nnz, const int32_t *pos, const int32_t *crd,
                                const float *vals, const float *B, int32_t k, int64_t ldb, float *C, int64_t ldc,
                                int32_t tile, int32_t over, int32_t chunk, bool plain, const Workspace &w, hipStream_t s, const int32_t *records);
hipError_t launch_spmm_rowsplit(int32_t rows, const int32_t *pos, const int32_t *crd, const float *vals,
                                const float *B, int32_t k, int64_t ldb, float *C, int64_t ldc,
                                hipStream_t s);

// BCSR (SpMV: bs = 4 has its own kernel, 2 and 8 share one; SpMM: bs in {2, 4, 8})
bool bcsr_tile_ok(int32_t tile);
bool bcsr_g_tile_ok(int32_t bs, int32_t tile);
hipError_t launch_spmv_bcsr_g_main(int32_t bs, int32_t brows, int32_t nblocks, const int32_t *pos, const int32_t *crd,
                                   const float *vals, const float *x, float *y, int32_t tile, const Workspace &w,
                                   hipStream_t s, int search);
hipError_t launch_spmv_bcsr4_main(int32_t brows, int32_t nblocks, const int32_t *pos, const int32_t *crd,
                                  const float *vals, const float *x, float *y, int32_t tile,
                                  const Workspace &w, hipStream_t s, int search);
// Rows of C that fill 64-byte pieces.
inline bool spmm_pieces(const float *C, int32_t k, int64_t ldc) { return k % 16 == 0 && ldc % 16 == 0 && (reinterpret_cast<uintptr_t>(C) & 63) == 0; }
// Rows of C that don't fill 64-byte pieces are stored through the L2 (spmm.hip has the reason) where rows have few blocks and C fits the memory-side cache, or most
// rows are empty.  Otherwise a wave per tile is slower than a workgroup where a row of C is all there is to do.  us workgroup / past the L2 / through it:
//   a block per row: 2 x 2, C 125 MB, k = 28 52 / 51 / 32;  206 MB, 45 60 / 72 / 43;  4 x 4, 130 MB, 28 62 / 67 / 41;  206 MB, 45 82 / 99 / 61;  240 MB, 50 80 / 100 / 89;  384 MB, 28
//   166 / 182 / -, 274 MB, 20 155 / 134 / -;  8 x 8, 206 MB, 45 91 / 93 / 110;  411 MB, 45 161 / 148 / -;  558 MB, 61 169 / 190 / -.  Two: 2 x 2, 28 42 / 27 / 24, 4 x 4, 45 56 / 54 / 44, 343 MB,
//   50 146 / 136 / -, 418 MB, 61 152 / 163 / -.  Three: 2 x 2, 28 41 / 22 / 23, 4 x 4, 45 54 / 43 / 44;  four: 2 x 2, 28 38 / 17 / 19.
//   a block in four rows: 4 x 4, 288 MB, 45 126 / 128 / 80;  in 16: 2 x 2, 580 MB 257 / 187 / 163
inline bool spmm_blocks_plain(int64_t brows, int64_t nblocks, int32_t bs, const float *C, int32_t k, int64_t ldc)
{
    return !spmm_pieces(C, k, ldc) && 2 * nblocks < 5 * brows && (brows * bs * ldc <= (int64_t(192) << 18) || 4 * nblocks < 3 * brows);
}
// Blocks: a wave per tile (spmm_blocks.hip, reads the table) or a workgroup, whose 64 lanes own one column each or more.  us workgroup / wave:
//   k = 8, 4 x 4, 1.8 M blocks 244 / 64;  8 x 8, 0.9 M 386 / 92;  2 x 2, 3.6 M 263 / 79;  k = 32 246 / 165, 400 / 196, 268 / 151;  48 262 / 227, 405 / 298, 271 / 224;
//   64: B 220 MB 300 / 308, 414 / 340, 290 / 307;  20 MB, 0.16 M blocks 34.8 / 31.5, 2 x 2, 0.8 M 67 / 59;  66 and more: 345 / 340, 517 / 511, 352 / 354, 200 921 / 1090
//   few tiles, where the workgroups' kernel searches its rows and saves a launch: 4 x 4, k = 8, 62 tiles 12.6 / 10.9;  8 x 8, 32 20.1 / 17.0; but 48 20.0 / 24.0
//     (4 x 4 12.9 / 13.8) and 2 x 2 9.6 / 11.0, up to 500 tiles 28.1 / 31.6 (13.9 / 14.1, 10.2 / 10.8), with 875 40.5 / 32.7 (19.3 / 16.2, 12.5 / 10.6);  a handful of blocks in less than a tile:
//     8 blocks of 4 x 4 6.4 / 7.2, 32 6.8 / 7.2, 48 8.4 / 7.1;  8 x 8, 16 7.4 / 7.9, 32 10.3 / 8.0
inline bool spmm_blocks_by_wave(int32_t bs, int64_t brows, int64_t bcols, int64_t nblocks, int32_t k, const float *C, int64_t ldc, int32_t tile)
{
    const int64_t ntiles = (nblocks + tile - 1) / tile;
    if (k < 4 || k > 64 || nblocks * bs <= 128 || (k > 48 && bs < 8 && bcols * bs * k > (int64_t(24) << 18)) || ntiles < (bs >= 4 && k <= 32 ? 1 : 600)) return false;
    if (spmm_pieces(C, k, ldc) || spmm_blocks_plain(brows, nblocks, bs, C, k, ldc)) return true;
    if (2 * nblocks < 3 * brows) return k <= (bs == 8 ? 32 : 24);
    return bs != 4 || k <= 40 || 2 * nblocks >= 5 * brows || (k <= 56 && bcols * bs * k <= (int64_t(24) << 18));
}
hipError_t launch_spmm_bcsr_wave(int32_t bs, int32_t brows, int32_t bcols, int32_t nblocks, const int32_t *pos, const int32_t *crd,
                                 const float *vals, const float *B, int32_t k, int64_t ldb, float *C, int64_t ldc, int32_t tile,
                                 int32_t over, const Workspace &w, hipStream_t s);
hipError_t launch_spmm_bcsr_main(int32_t bs, int32_t brows, int32_t bcols, int32_t nblocks, const int32_t *pos, const int32_t *crd,
                                  const float *vals, const float *B, int32_t k, int64_t ldb, float *C,
                                  int64_t ldc, int32_t tile, const Workspace &w, hipStream_t s, int search);

// Column-slab hierarchy of a CSR matrix (slab.hip)
constexpr int32_t kSlabCols = 32736;        // columns per slab: 32 * 1023 floats = 127.9 KB of x in LDS (15-bit in-slab column)
constexpr int32_t kSlabColsF64 = 16352;     // fp64: 127.75 KB of x next to 32 KB of pair sums (16 waves x 256 doubles)
constexpr int32_t kSlabChunk = 512;         // slots per chunk (one wave: 8 per lane)
constexpr int32_t kSlabBuildBlock = 2048;   // CSR positions per block of the bucketing kernels
constexpr int32_t kSlabMaxSlabs = 8192;     // the bucketing kernels keep one counter per slab in LDS
constexpr int32_t kSlabTile = 2048;         // position tile of the second step (pairs per workgroup)
constexpr int32_t kSlabTileF64 = 1024;      // the same for fp64 (its tile kernel holds twice the LDS per position)
inline int64_t slab_max_slots(int64_t cols, int64_t nnz, int32_t W)
{
    const int64_t S = (cols + W - 1) / W;
    const int64_t padded = nnz + S * (kSlabChunk - 1);
    return (padded + kSlabChunk - 1) / kSlabChunk * kSlabChunk;
}
constexpr int32_t kStageSlabs = 256;        // up to this many slabs the analysis works block by block (k_block_place)
struct SlabBuildSpace {
    int32_t *meta, *tile_row, *H, *src;
    int32_t *srow, *F, *mark, *pair_at, *scan_tmp;                      // more than kStageSlabs slabs
    int32_t *total, *part;                                              // at most kStageSlabs slabs
    uint16_t *H16, *N16, *pbits_pre;
    unsigned long long *pbits, *chunk_at;
    size_t bytes;
};
size_t scan_tmp_ints(int64_t n);
SlabBuildSpace carve_slab_build(void *base, int64_t rows, int64_t cols, int64_t nnz, int32_t W);
hipError_t launch_slab_build(int32_t rows, int32_t cols, int32_t nnz, const int32_t *pos, const int32_t *crd,
                             const float *vals, const SlabBuildSpace &w, float *svals, uint16_t *scol,
                             int32_t *chunk_pair, int32_t *slab_chunk, int32_t *qpos, int32_t *qidx, int32_t qtile,
                             int32_t *qtile_row, hipStream_t s);
hipError_t launch_slab_build_f64(int32_t rows, int32_t cols, int32_t nnz, const int32_t *pos, const int32_t *crd,
                                 const double *vals, const SlabBuildSpace &w, double *svals, uint16_t *scol,
                                 int32_t *chunk_pair, int32_t *slab_chunk, int32_t *qpos, int32_t *qidx, int32_t qtile,
                             int32_t *qtile_row, hipStream_t s);
hipError_t launch_slab_pairs_f64(const double *svals, const uint16_t *scol, const int32_t *chunk_pair,
                                 const int32_t *slab_chunk, const double *x, double *P, int32_t cols, int32_t nslabs,
                                 int32_t nchunks, int32_t nwg, hipStream_t s);
hipError_t launch_slab_pairs(const float *svals, const uint16_t *scol, const int32_t *chunk_pair,
                             const int32_t *slab_chunk, const float *x, float *P, int32_t cols, int32_t nslabs,
                             int32_t nchunks, int32_t nwg, hipStream_t s);
hipError_t launch_fill_int(int32_t *p, int64_t n, int32_t v, hipStream_t s);
// y = Q * P with unit values: the tile kernel of the CSR SpMV without the load of vals (tile 2048)
hipError_t launch_spmv_csr_ones(int32_t rows, int32_t cols, int32_t nnz, const int32_t *pos, const int32_t *crd,
                                const float *x, float *y, const Workspace &w, hipStream_t s);
hipError_t launch_spmv_csr_f64_ones(int32_t rows, int32_t nnz, const int32_t *pos, const int32_t *crd, const double *x,
                                    double *y, int32_t tile, const Workspace &w, hipStream_t s);

#ifdef PSK_CU_TRACE
hipError_t cu_trace_set_spmv_csr(void *buf, unsigned records);
hipError_t cu_trace_set_slab(void *buf, unsigned records);
#endif

// MTTKRP on a three-level hierarchy
bool mttkrp_tile_ok(int32_t tile);
hipError_t launch_partition_csf3(int32_t nslices, int32_t nfibers, int32_t nnz, const int32_t *pos_k,
                                 const int32_t *pos_l, int32_t tile, int32_t *tile_slice, int32_t *tile_fiber,
                                 hipStream_t s);
hipError_t launch_mttkrp_main(int64_t dim_k, int64_t dim_l, int32_t nslices, int32_t nnz, const int32_t *crd_i, const int32_t *pos_k,
                              const int32_t *crd_k, const int32_t *pos_l, const int32_t *crd_l, const float *vals,
                              const float *C, int64_t ldc, const float *D, int64_t ldd, int32_t j, float *A,
                              int64_t lda, int32_t tile, const Workspace &w, const int32_t *tile_fiber,
                              hipStream_t s);

}  // namespace psk
