// CSR SpMM for dense operands of up to 128 columns.  The wide SpMM kernel maps the 64 lanes of a wave to 64*VEC columns of
// B and takes one position per step; with few columns most of its instructions are spent on book-keeping per position.
// Here a lane owns VEC = 4 adjacent columns and the wave is split into G groups of 64/G lanes that take G consecutive
// positions in one step, so that one 16-byte load per lane fetches G rows of B.  Every lane keeps the partial sums of its
// group for the open row; at a row end the sums of the groups are added across the wave.  Cut, row-end flags, records and
// carries: as in the wide kernel.
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

}  // namespace psk
