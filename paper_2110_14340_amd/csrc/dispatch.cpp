// Loop-kind dispatch, default launch configurations and their validation.
#include "jacc.h"
#include "kernels.h"

namespace jk {

static int64_t inner_extent(const Launch &L) {
    // length of the contiguous (innermost) dimension of the first argument
    int nd = 1;
    for (int i = 1; i < 4; ++i)
        if (L.ext[i] > 0) nd = i + 1;
    return L.ext[nd - 1];
}

// The heat kernels' multi-row shape: threads, rows and planes a wave, and the
// order of the tiles.  Times are us a step, in a graph.
static Cfg heat_shape(const Launch &L, Cfg c) {
    const int64_t cells = array_bytes(L) / 8;
    const int64_t lanes = (L.ext[2] + c.vec - 1) / c.vec;
    auto set = [&](int bx, int by, int tile, int rows, int order) {
        c.bx = bx;
        c.by = by;
        c.tile = tile;
        c.rows = rows;
        c.order = order;
        return c;
    };
    // 128x2 threads read a row in longer runs (95x131x203: 11.3, 14.1 as 64x4)
    // unless that idles more lanes (300^3: 128 and 100)
    const bool wide = (lanes + 127) / 128 * 128 == (lanes + 63) / 64 * 64;
    if (cache_resident(L)) {
        // bound by waves in flight before bytes: small tiles (64^3: 6.0 as
        // 64x2x2 planes, 14 with 4 rows and 8 planes; 128^3 9.0 and 15.3),
        // y-blocked bricks so that a tile's neighbours run on the same XCD
        // (256^3: 43, 51 in row-major order).  Several partitions in one launch
        // take 4 rows a wave (256^3 over 4: 59, 66 with 2; 128^3 11.7 and 11.3).
        if (cells < (1 << 19)) return set(64, 2, 2, 2, 3);
        const bool split = 3 * L.part_rows < 2 * L.ext[0] && cells >= (1 << 22);
        return wide ? set(128, 2, 3, split ? 4 : 2, 3) : set(64, 4, 3, split ? 4 : 2, 3);
    }
    // bound by HBM: 4 rows and 8 planes re-read the least.  A row held by one
    // workgroup (up to 256 lanes) streams best in row-major order from 256x1
    // threads (300x300x386: 124, 137 as 64x4; 400^3 213 and 232; 175x435x501 131,
    // 143 as bricks), except full ones, whose power-of-two strides prefer 128x2
    // (300x400x512: 192, 199 as 256x1), in bricks where two planes fill an XCD's
    // L2 (512^3: 394, 408 as 256x1; 512x512x510 418 and 435; 300x400x510 214 in
    // bricks, 202 in row-major order).  Other rows: 128x2 where it idles no
    // lanes and a row fits (700x700x200: 312, 356 as 64x4), 64x4 elsewhere
    // (300^3: 97, 123 as 128x2; 60x1000x1400: 255 and 276).
    if (lanes > 253 && lanes <= 256)
        return 8 * L.ext[1] * L.ext[2] > 2000000 ? set(128, 2, 4, 4, 3) : set(128, 2, 8, 4, 1);
    if (lanes > 192 && lanes <= 256) return set(256, 1, 8, 4, 1);
    if (lanes <= 128 && wide) return set(128, 2, 4, 4, 1);
    return set(64, 4, 8, 4, 1);
}

Cfg default_config(int kind, const Launch &L, Cfg c) {
    const bool odd = inner_extent(L) % 2 != 0;
    switch (kind) {
        case JACC_LOOP_JACOBI2D: {
            if (!c.vec) {
                c.vec = 2;
                c.odd = odd;
            }
            if (!c.march) c.march = 2;
            if (!c.rows) c.rows = 1;
            if (c.persistent) {  // tiles of 256 threads along a row
                if (!c.bx) c.bx = 256;
                if (!c.by) c.by = 1;
                if (!c.tile) c.tile = 4;
                if (!c.order) c.order = 1;
                break;
            }
            // Beyond the cache: 64x4 threads, whose waves share the rows beside
            // theirs within the workgroup, in rows of whole 64-byte pieces (us a
            // sweep of 2^26 cells as 256x1 and 64x4: 3696 columns 185 and 170, 5744
            // 188 and 170, 11888 183 and 170); in other rows a tile's ends are
            // parts of lines that two workgroups touch, and 256x1 has fewer ends
            // (4306 columns 177 and 187, 6556 175 and 185, 12700 175 and 194).  256x1
            // also in rows of 4096 columns or a multiple, where the tile below runs
            // on the same XCD (8192^2: 171 and 174), and from 2^16 columns on
            // (33x3000000: 257 and 270).  Column slabs, whose pitch is their own:
            // 64x4 unless the tile below runs on the same XCD (10001x6001 over 8: 178,
            // 196 as 256x1).
            const bool cached = cache_resident(L);
            const int64_t cells = array_bytes(L) / 8;
            // under 4096 cells a step is its launch, and the shape stays
            // 256x1 of 4 rows, as loop records report it (60x60 in a graph: 3.6
            // us, 2.9 as 64x4 of 1)
            const bool tiny = cells < 4096;
            const int64_t nx = L.ext[1];
            const bool along = tiny || (!cached && (L.part_dim == 1 ? (nx + 511) / 512 % 8 == 0
                                                                    : nx % 8 != 0 || nx % 4096 == 0 || nx >= (1 << 16)));
            // short tiles while there are few of them (512^2: 3.9 us with 2
            // rows, 4.3 with 4, 5.4 with 8; 2048^2: 12.3 with 4, 11.9 with 8)
            // (several partitions in a launch: 4, 1175x780 over 8 8.5 us, 8.9 with 2)
            const bool split = 3 * L.part_rows < 2 * L.ext[0];
            const int tile = c.tile ? c.tile : !cached || tiny ? 4 : cells < (1 << 20) && !split ? 2 : cells < (1 << 22) ? 4 : 8;
            c.tile = tile;
            if (!c.bx && !c.by && !along) {
                // no more row groups than a partition's rows fill (us a sweep as
                // 64x4 and so: 8x1000000 over 4 partitions 62 and 28, 10x500000 over
                // 4 34 and 18, 20x300000 over 2 19.4 and 17.3)
                const int64_t groups = (L.part_rows + tile - 1) / tile;
                c.by = groups <= 1 ? 1 : groups == 2 ? 2 : 4;
                c.bx = 256 / c.by;
            }
            if (!c.bx) c.bx = 256;
            if (!c.by) c.by = 1;
            if (!c.order) c.order = cached ? 2 : 1;
            break;
        }
        case JACC_LOOP_HEAT3D: {
            if (!c.vec) {
                c.vec = 2;
                c.odd = odd;
            }
            if (!c.march) c.march = 2;
            const Cfg given = c;
            if (!c.rows) {  // multi-row waves need workgroups of at most 256 threads
                const int bx = c.bx ? c.bx : 128, by = c.by ? c.by : 2;
                if (c.persistent || bx * by > 256) c.rows = 1;
            }
            if (c.rows == 1) {
                if (!c.bx) c.bx = 256;
                if (!c.by) c.by = 4;
                if (!c.tile) c.tile = 4;
                if (!c.order) c.order = 1;
                break;
            }
            const Cfg d = heat_shape(L, c);
            if (!c.bx && !c.by) {
                // no more row groups than the field's rows fill: with a residual
                // the waves without rows wait for the others' sums (3000x3x3000
                // 111 us a step as 64x4, 4x4x1000000 41 as 128x2)
                const int rows = c.rows ? c.rows : d.rows;
                const int64_t groups = (L.ext[1] - 2 + rows - 1) / rows;
                c.by = groups <= 1 ? 1 : groups == 2 && d.by > 2 ? 2 : d.by;
                c.bx = d.bx * d.by / c.by;
            }
            if (!c.bx) c.bx = 128;
            if (!c.by) c.by = 2;
            if (!c.rows) c.rows = d.rows;
            if (!c.tile) c.tile = d.tile;
            if (!c.order) c.order = d.order;
            // a residual takes one partial sum per workgroup: fields with more
            // workgroups than half the partial buffer take 128x2 threads, 4 rows
            // and 8 planes, which serve every field that fits at all
            const int64_t wgs = ((L.ext[2] + (int64_t)c.bx * c.vec - 1) / ((int64_t)c.bx * c.vec)) *
                                ((L.ext[1] + (int64_t)c.by * c.rows - 1) / ((int64_t)c.by * c.rows)) *
                                ((L.ext[0] + c.tile - 1) / c.tile);
            if (wgs > kWgCapacity / 2) {
                c.bx = given.bx ? given.bx : 128;
                c.by = given.by ? given.by : 2;
                c.rows = given.rows ? given.rows : 4;
                c.tile = given.tile ? given.tile : 8;
                c.order = given.order ? given.order : 3;
            }
            break;
        }
        default:
            if (!c.bx) c.bx = 256;
            if (!c.by) c.by = 1;
            // SpMV: non-temporal col/val loads; the runtime sets the lanes per
            // row by the matrix's mean row length
            if (!c.tile) c.tile = kind == JACC_LOOP_GEMM ? 16 : kind == JACC_LOOP_SPMV_CSR ? 16 : 1;
            if (!c.vec) c.vec = 1;
            if (!c.order) c.order = kind == JACC_LOOP_SPMV_CSR ? 2 : 1;
            if (!c.march) c.march = 1;
            if (!c.rows) c.rows = 1;
            break;
    }
    return c;
}

int check_config(const Launch &L) {
    const Cfg &c = L.cfg;
    if (c.persistent != 0 && c.persistent != 1) return 1;
    if (c.persistent && L.kind != JACC_LOOP_JACOBI2D && L.kind != JACC_LOOP_HEAT3D) return 1;
    switch (L.kind) {
        case JACC_LOOP_JACOBI2D:
        case JACC_LOOP_HEAT3D:
            if (c.bx < 64 || c.bx % 64 || c.by < 1 || c.bx * c.by > 1024) return 1;
            if (c.tile < 1 || c.tile > 65536) return 1;
            if (c.vec != 1 && c.vec != 2) return 1;
            if (c.vec == 2 && inner_extent(L) % 2 && !c.odd) return 1;
            if (c.order != 1 && c.order != 2 && (c.order != 3 || L.kind != JACC_LOOP_HEAT3D)) return 1;
            if (c.march != 1 && c.march != 2) return 1;
            if (c.rows != 1 && (L.kind != JACC_LOOP_HEAT3D || c.persistent)) return 1;
            if (c.rows != 1 && c.rows != 2 && c.rows != 4 && c.rows != 8) return 1;
            if (c.rows != 1 && c.bx * c.by > 256) return 1;  // multi-row waves: workgroups of at most 256
            return 0;
        case JACC_LOOP_GEMM:
            // the values earlier kernels took; the kernel chooses its tile by shape
            return ((c.tile == 16 || c.tile == 32) && (c.bx == 256 || c.bx == 512)) ? 0 : 1;
        case JACC_LOOP_SPMV_CSR:
            // order 4: the binned form; tile, by and rows take the values that
            // an earlier form split its work by, without effect
            if (c.order == 4)
                return ((c.tile == 1 || c.tile == 2 || c.tile == 4 || c.tile == 8 || c.tile == 16) &&
                        (c.by == 1 || c.by == 2 || c.by == 4 || c.by == 8) &&
                        (c.rows == 1 || (c.tile == 1 && (c.rows == 2 || c.rows == 4))))
                           ? 0
                           : 1;
            if (c.tile != 4 && c.tile != 8 && c.tile != 16) return 1;
            return (c.order == 1 || c.order == 2) ? 0 : 1;
        case JACC_LOOP_SUM:
        case JACC_LOOP_SCATTER_SQ:
        case JACC_LOOP_PRED_CHAIN:
            return 0;  // fixed internal configurations; fields are ignored
        default:
            return 1;
    }
}

int64_t reduction_workgroups(const Launch &L) {
    switch (L.kind) {
        case JACC_LOOP_HEAT3D: return heat3d_workgroups(L);
        case JACC_LOOP_SUM: return sum_workgroups(L);
        default: return 0;
    }
}

hipError_t launch_loop(const Launch &L, hipStream_t s) {
    switch (L.kind) {
        case JACC_LOOP_JACOBI2D: return launch_jacobi2d(L, s);
        case JACC_LOOP_HEAT3D: {
            hipError_t e = launch_heat3d(L, s);
            if (e != hipSuccess || !L.wg_partials) return e;
            return launch_result(L, heat3d_workgroups(L), s);
        }
        case JACC_LOOP_SUM: return launch_sum(L, s);
        case JACC_LOOP_GEMM: return launch_gemm(L, s);
        case JACC_LOOP_SPMV_CSR: return launch_spmv(L, s);
        case JACC_LOOP_SCATTER_SQ: return launch_scatter(L, s);
        case JACC_LOOP_PRED_CHAIN: return launch_chain(L, s);
        default: return hipErrorInvalidValue;
    }
}

}  // namespace jk
