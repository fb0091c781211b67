// Chooses the kernel, the row slicing and the launch shape for one layer
// application and sizes its workspace.
#include <algorithm>
#include <cstdio>
#include <cstdlib>

#include "pivot_frag.h"

namespace pivot {

// Compute units of the current device (asked once per device).
static int device_cus() {
    static int cus[16] = {};
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess) { (void)hipGetLastError(); return 1; }
    int& c = cus[dev & 15];
    if (c == 0) {
        int n = 0;
        if (hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) == hipSuccess && n > 0) c = n;
        else { (void)hipGetLastError(); c = 1; }
    }
    return c;
}

// Batch rows the LDS-fed matrix-core kernel stages: 4, or 8 (batch 9..16 then runs as two launch rows of 8, each
// workgroup gathering half the rows: staging all 16 in one workgroup was measured slower at every density, 6.0 ->
// 4.7 us at 5 % kept and 13.4 -> 12.3 at 50 % on 4096x4096, where 16 rows no longer fit; four launch rows of 4
// were slower again from 10 % kept on: the weights are then streamed four times).
static int mfma_lds_rows(int batch) { return batch <= 4 ? 4 : 8; }

// Tiles per wavefront whose block columns fit the batched matrix-core kernel's registers (64 each, frag_cols), less
// one group of tiles for the rounding of the split over wavefronts.
static int frag_wave_tiles(const FcShape& s) { return frag_cols(s.bw, 16 / elem_size(s.wdtype)) * 64 - 8; }

static void frag_split(const FcShape& s, int batch, int* slices, int* blocks);

// fp32, batch 2-8, x in block order: whether the vector kernel is ahead.  It streams the weights once per 4 batch rows
// (twice at batch 5-8) but cuts a block row down to slices of 4 rows, where the fragment form stops at 16: with fewer
// work items than compute units and long ones the fragment form leaves the chip idle.  Us for a layer behind one of 64
// inputs, vector / fragment form, batch 2, 4, 8 (columns per work item; items of 16 rows):
//   4096 -> 1000, 32x32, 50 % (2048; 64)   7.6 / 10.0    8.5 / 10.4   8.8 / 10.7
//   3000 -> 1000, 16x64, 50 % (1536; 63)   7.6 / 9.1     8.2 / 9.5    9.8 / 10.0
//   3000 -> 1000, 32x64, 10 % (320; 64)    6.6 / 7.0     7.3 / 7.3    7.8 / 7.8
//   4096 -> 1000, 16x64, 25 % (1024; 63)   7.1 / 7.7     7.8 / 8.1    9.1 / 8.4
//   1000 -> 1000, 64x64, 50 % (512; 64)    7.0 / 6.9     7.9 / 7.3
//   3000 -> 4096, 32x32, 25 % (768; 256)   8.3 / 8.2     9.2 / 8.7   10.5 / 9.3
//   9000 -> 8000, 16x32, 10 % (896; 500)  10.8 / 11.2   11.8 / 11.6  16.8 / 12.6
//   4096 -> 8000, 8x32, 5 % (192; 1000)    7.6 / 8.8     8.1 / 9.1   10.7 / 9.9
//   9000 -> 1000, 16x16, 25 % (2256; 63)   8.9 / 9.8    10.0 / 10.2  13.1 / 11.9
//   9000 -> 2000, 16x16, 25 % (2256; 125) 10.3 / 9.9    11.3 / 10.2
//   4096 -> 2000, 8x8, 50 % (2048; 250)    9.4 / 10.0   10.7 / 10.3
// Of tiles up to 16 columns wide a step of the fragment form is at most one tile and it is ahead but for the longest.
static bool block_order_vector(const FcShape& s, int batch) {
    int slices, blocks;
    frag_split(s, batch, &slices, &blocks);
    const long long items = (long long)s.nchunks * slices;
    const int cols = s.mean_tiles * s.bw;                // per work item
    if (batch > 4) return s.bw >= 32 && ((cols >= 750 && items <= 32) || (cols >= 1400 && items <= 64));
    if (s.bw < 32) return (cols >= 1400 && items <= 64) || (s.bh == 8 && batch == 2 && cols >= 1000);
    if (items < 256) return cols >= (batch == 2 ? 200 : 700);
    return items >= 500 && (s.bh == 8 || (batch == 2 && cols >= 400));
}

// Row slices <= want of whole MFMA row blocks: 16 rows (tiles 16 columns wide are then taken in pairs) or 32.
static int mfma_slices(const FcShape& s, int want) {
    const int mr = (mfma_kind(s.wdtype, s.bh, s.bw) == 0 || s.bw == 16) ? 16 : 32;
    int sl = want < 1 ? 1 : want;
    while (sl > 1 && (s.bh % sl != 0 || (s.bh / sl) % mr != 0)) sl /= 2;
    return sl;
}

// Which kernel applies the layer:
//   kPathVector    batch 1-2 (and whatever the others do not take): FMA / dot2 against x staged in LDS, launch rows of
//                  at most 4 batch rows
//   kPathFrag      both types, every tile shape: MFMA with the B fragments read from an x in fragment order, the
//                  weights streamed once for up to 64 batch rows; a natural-order x is copied by a launch of its own
//   kPathMfmaLds   fp16, batch >= 3: MFMA with the B fragments read from x staged in LDS (4 or 8 batch rows per launch row)
//   kPathMfmaXrow  fp16, batch 5 on, rows of at most 4096 columns: MFMA with the B fragments gathered from a copy of the rows of x in LDS
// An x that the layer or cell before produced (kXBlock) arrives in the order the kernel wants, so from batch 2 on the
// fragment form has nothing to pay for and streams the weights once (three fp16 layers of 25088-4096-4096-1000
// at 10 % kept, batch 32: 23.1 us with the LDS-fed form behind the boundaries, 17.9 with this one).  (fp32 layers of up to
// 8 batch rows: block_order_vector.)  For an x from the
// caller the copy costs about 2.2 us and a second launch, and the other forms repeat work per launch row instead:
// - fp32, and fp16 tiles no other matrix-core form takes: the vector kernel streams the weights, LDS-bound at 2-5.5
//   TB/s, once per 4 batch rows.  4096x9216 fp32, 10 % kept (15 MB), vector / fragment form, batch 2: 6.6 / 9.3 us, 4:
//   8.9 / 7.9, 8: 13.5 / 9.3, 16: 20.5 / 8.8, 64: 64.6 / 17.2; 2048x2048, 25 % (4 MB), batch 8: 4.8 / 6.1, 16: 7.5 /
//   6.4; 1000x4000, 10 % (1.6 MB), batch 16: 6.0 / 5.7, 64: 15.9 / 7.4; 1000x1000, 25 % (1 MB), batch 64: 5.9 / 6.1.
//   So from 12 MB of repeated weights on (14 MB of weights where one launch row covers batch 3-4).
// - fp16 tiles that fit an MFMA shape: the LDS-fed form gathers the x-segments of its work items anew in every launch
//   row of 8.  LDS-fed / fragment form, batch 16: 8192x8192, 25 % (524 K columns staged per launch row) 15.7 / 12.2 us,
//   10 % (210 K) 10.6 / 9.5, 4096x9216, 10 % (118 K) 8.4 / 7.6, 4096x4096, 10 % (52 K) 5.5 / 5.6 and at batch 32 8.4 /
//   6.8, 64x16 tiles (26 K) at batch 32 6.05 / 6.9 and at batch 64 9.5 / 9.1.  So from 100 K restaged columns on.
// The LDS-fed form gathers through the plan's source-ordered lists and is taken while its staged rows fit in 48 KB.
// At batch 9-16 its staging (16 rows x staged columns two-byte gathers per work item, repeated by every row slice)
// bounds it; gathering where the fragment is formed needs one copy of x per work item instead, whatever the number of
// staged columns.  The copy costs a work item 1.5-2.3 us (4096 columns: 128 KB through one compute unit's memory
// pipeline before its first MFMA), the gathers 0.2-0.9 us, so the x-row form is taken from a quarter of the columns
// staged per work item on (4096x4096, 64x16 tiles, batch 16, cold: 8.3 -> 7.1 us at 25 % kept, 12.5 -> 9.1 at 50 %, 14.9
// -> 12.7 dense; at 10 % it would lose, 6.0 -> 6.3, at 5 % 4.8 -> 6.3).  Batch 5-8 takes it under the same rule (only
// the rows that exist are copied; same matrix, batch 8: 6.5 -> 6.1 us at 25 %, 9.65 -> 8.1 at 50 %, 12.45 -> 11.7 dense,
// batch 5 the same within 0.1 us); at batch 4 it loses (5.6 -> 6.0, 7.7 -> 7.9, 9.8 -> 11.1).  The fragment form is
// 0.5-1 us behind it (batch 16: 6.2 / 7.0 at 25 %, 8.4 / 8.8 at 50 %, 11.7 / 12.6 dense).
int fc_path(const FcShape& s, int batch) {
    const int layout = s.layout, wdtype = s.wdtype, bh = s.bh, bw = s.bw, lds_tiles = s.lds_tiles;
    // the matrix-core kernels read A fragments from row-major (BRC) tiles only
    if (layout != PIVOT_BRC || batch < 2) return kPathVector;
    const bool frag = s.x_from != kXNoCopy && (long long)s.xrow_len * batch * elem_size(wdtype) < (1ll << 31);
    const double weight_mb = (double)s.nchunks * s.mean_tiles * bh * bw * elem_size(wdtype) * 1e-6;
    if (frag && s.x_from == kXBlock) {
        const bool vector = wdtype == PIVOT_F32 && batch <= 8 && block_order_vector(s, batch);
        return vector ? kPathVector : kPathFrag;
    }
    if (mfma_kind(wdtype, bh, bw) < 0) {
        const int launch_rows = (batch + 3) / 4;
        return frag && batch >= 3 && (launch_rows > 1 ? (launch_rows - 1) * weight_mb >= 12.0 : weight_mb >= 14.0) ? kPathFrag : kPathVector;
    }
    if (batch < 3) return kPathVector;
    bool lds = false;
    if (lds_tiles > 0) {
        const int rows = mfma_lds_rows(batch);
        const size_t xs_bytes = (size_t)rows * ((size_t)lds_tiles * bw + 8 + 16) * 2;   // + the paired form's zeroed columns
        // every launch row of 8 batch rows streams the weights again and gathers its own rows: beyond two launch
        // rows the form is kept while the launch rows together stage at most 5120 columns per work item
        // (4096x4096, 64x16 tiles, against the fragment form: batch 24 at 5 % kept 6.2 -> 5.1 us, batch 64 8.7 -> 7.8)
        const size_t launch_rows = (size_t)(batch + rows - 1) / rows;
        const bool restage = frag && (double)(launch_rows - 1) * s.nchunks * s.mean_tiles * bw >= 100e3;
        lds = !restage && xs_bytes <= 48 * 1024 && (launch_rows <= 2 || launch_rows * lds_tiles * bw <= 5120);
    }
    if (batch >= 5 && s.xrow_len > 0 && s.chunk_tiles > 0) {
        // 16 rows of x (each with 16 zeroed bytes behind it) and the work item's gather indices in LDS; a lane
        // copies at most 8 vectors of a row, a thread at most 4 int4 of indices
        const size_t vecs = ((size_t)s.xrow_len + 7) / 8;
        const size_t cols = ((size_t)s.chunk_tiles + 1) * bw;
        const size_t copy_bytes = (size_t)16 * xrow_bytes((int)vecs) + cols * 4;
        const long long items = (long long)s.nchunks * mfma_slices(s, s.row_slices) * ((batch + 15) / 16);
        // "a quarter of the columns staged per work item": at batch 5-8 of the AVERAGE work item.  With a few long block
        // rows among many short ones most work items copy all of x for a handful of tiles, which the 8-row LDS-fed form
        // does not (4096x4096, per-row counts from 96 down to 2: the copy loses at batch 16 and wins at batch 5-8; batch
        // 9-16 keeps the rule it was measured with).
        const bool quarter = (batch <= 8 ? ((size_t)s.mean_tiles + 1) * bw : cols) * 4 >= (size_t)s.xrow_len;
        bool pays;
        if (lds && s.xrow_len <= 2048) {
            // Rows of at most 2048 columns against the LDS-fed form.  Rows that are whole aligned vectors pay for their copy
            // from an eighth of them staged per work item on, while the work items of the launch run beside each other: two
            // per compute unit, of tiles 64 columns wide one (their time steps from 257 on, 4.1 -> 5.7 us, of tiles 32 wide
            // at 513; registers and LDS would hold two of either, why the wide ones do not gain is not known.  The 256 is a
            // literal so that a plan made without a device names the same kernel).  LDS-fed / this one, us: 784 columns,
            // 32x32 tiles, batch 16, 156 items 4.7 / 3.9; 1520, 32x32, batch 24, 344 items 6.4 / 5.5; 744, 16x64, batch 64,
            // 212 items 5.8 / 4.5; 760, 64x64, batch 24, 304 items 4.6 / 6.8; 256 staged of 1512, 16x32, batch 6, 627 items
            // 5.4 / 6.4; 64 staged of 800, 32x64, batch 16 3.6 / 4.2.  Rows that are not cost it 0.3-0.5 us more and the
            // LDS-fed form, which gathers them from memory, nothing (729 columns, 32x16, batch 8 3.1 / 4.1; 713, 64x16,
            // batch 64 3.4 / 4.4; 795, 64x32, batch 24 3.5 / 4.0).
            // Whatever the rows, at batch 5-16 one copy of 16 rows is ahead where the gathers bound the LDS-fed form, which
            // come again with every row slice and launch row of 8: from 200 K columns staged by all its work items on, 120 K
            // where it has two launch rows, while this form has at most 512 work items, and from 1024 columns staged by one of
            // at most 256 on (1481 columns, 32x64, batch 16, 284 items of 1152 7.4 / 5.1; 1284, 64x64, batch 16, 668 of 202
            // 10.4 / 8.1; 752, 64x64, batch 9, 548 of 276 9.9 / 6.3; 1493, 32x64, batch 16, 364 of 332 5.5 / 4.6; but 1727,
            // 16x64, batch 16, 576 of 256 6.3 / 7.2; of more than 512 work items, whose partial sums of 16 rows also take twice
            // the scratch, batch 5-8 lost 1.2x in the mean, up to 1.5x).
            // Of 2400 drawn layers with rows of both kinds the rule is 0.6 % from the better form in the mean.
            const int slices = mfma_slices(s, batch > 8 && s.row_slices > 2 ? 2 : s.row_slices), launch_rows = batch > 8 ? (batch + 7) / 8 : 1;
            const double staged = (double)s.nchunks * slices * launch_rows * s.mean_tiles * bw;
            pays = (s.x_vec && (size_t)s.chunk_tiles * bw * 8 >= (size_t)s.xrow_len && items <= (bw == 64 ? 256 : 512)) ||
                   (batch <= 16 && ((staged >= (batch > 8 ? 120e3 : 200e3) && items <= 512) || (items <= 256 && s.chunk_tiles * bw >= 1024)));
        } else if (batch <= 16) {
            pays = quarter;
        } else {
            // Against the fragment form and its copy of x: two to four launch rows are ahead while they stage at most 2048
            // columns per work item and every item has a compute unit to itself, of rows up to 2048 columns half of one
            // (us, fragment form / this one: 300x1800 16x64 50 % batch 32 5.6 / 4.6; batch 64, 16x32 tiles: 1000x4090 25 %
            // 7.5 / 7.0, 1000x4096 50 % (2048 columns) 8.6 / 8.4, 300x4000 64x64 50 % 8.3 / 6.8; with more work items,
            // 8000x1000 32x32 20 %, batch 32 7.5 / 9.1, 2000x4090 32x32 25 % 9.7 / 12.3; with longer ones, 129x3594 rows by a
            // Zipf law 6.8 / 8.0; 64 columns wide, 3724x2024 16x64 7 % batch 32, 466 items 6.35 / 7.5, 1710x1128 22 % batch 64,
            // 428 items 6.3 / 7.4, 364 items 0.97x); of longer rows at batch 17-32 they are not (250x4090 25 % 4.9 / 5.3).
            pays = !lds && cols <= 2048 + (size_t)bw && (s.xrow_len <= 2048 ? items < (bw == 64 ? 384 : 512) : batch > 32 && items <= 256);
        }
        if (vecs <= 512 && cols <= 8192 && copy_bytes <= 156 * 1024 && pays) return kPathMfmaXrow;
    }
    if (lds) return kPathMfmaLds;
    return frag && batch >= 8 ? kPathFrag : kPathVector;
}

bool fc_wants_frag(const FcShape& s, int batch) { return fc_path(s, batch) == kPathFrag; }

// Row slices and blocks of 16 batch rows per launch row of the batched matrix-core kernel: slices of at most 32
// rows and the whole batch in one launch row (the weights stream once) where that gives a work item to every
// compute unit, else slices down to 16 rows (each reads the x of the whole block row), then shorter launch rows (each
// streams the weights).  Us per call with 32- / 16-row slices: 8192x8192 fp32 25 % kept, batch 64 (256 block rows)
// 33.0 / 37.4, 4096x25088 fp16 10 %, batch 4 (128 block rows) 9.15 / 8.8; with 1 / 2 / 4 blocks per launch row:
// 8192x8192 fp16, batch 64 26.9 / 20.0 / 17.5, 1000x4096 fp16 16x32 tiles (63 block rows), batch 64 7.55 / 7.56 / 8.8.
static void frag_split(const FcShape& s, int batch, int* slices, int* blocks) {
    int sl = s.bh > 32 ? s.bh / 32 : 1;
    const int need = (batch + 15) / 16;
    int nbt = s.x_from == kXNaturalRows16 ? 1 : (need > 2 ? 4 : need);
    auto items = [&]() { return (long long)s.nchunks * sl * ((need + nbt - 1) / nbt); };
    while (items() < 256 && s.bh / sl > 16) sl *= 2;
    while (items() < 256 && nbt > 1) nbt /= 2;
    *slices = sl;
    *blocks = nbt;
}

// Wavefronts per work item of the batched matrix-core kernel.  Each keeps up to 8 KB of weights and the x that goes with
// them in flight, so four fill a compute unit's queue, and several small workgroups per compute unit overlap one's
// epilogue with another's loads (us per layer call, 8 / 4 / 2 wavefronts: 4096x1024 fp16 8x8 tiles, batch 32
// 11.4 / 8.0 / 6.9; 4096x9216 fp32 10 % kept, batch 32 13.6 / 12.4 / 14.7; 8192x8192 fp16 25 % kept, batch 64
// 19.1 / 17.6 / 18.9; 16384x16384 fp16 64x64 tiles 10 % kept, batch 8 22.1 / 19.4 / 17.6): two with fp16 weights
// from two work items per compute unit on, and two where the work item has no more steps than two wavefronts request
// at once: the other two would only load copies and wait (a layer behind one of 64 inputs, us, 4 / 2 wavefronts: 300 ->
// 8000 fp32 8x32, 5 % kept, batch 6 11.1 / 8.6; 700 -> 8000 fp32 32x32, 10 %, batch 2 7.6 / 6.6; 700 -> 8000 fp16 32x64,
// 10 %, batch 4 7.7 / 6.7; 1000 -> 500 fp16 32x32, 5 %, batch 4 5.9 / 5.7), up to 16 steps at batch 2-8 and up to 8 beyond
// (fp32: to batch 16), where a step's x is heavier too (4096x3000 fp32 8x32, 5 %, 5 steps, batch 64 12.2 / 12.8; 1000x2048 fp16 16x32, 25 %, 16 steps, batch 64 5.6 / 5.8; 4096 -> 2048 -> 2000 fp16 8x8,
// 20 %, 6 steps, batch 64 13.2 / 12.1).
static int frag_waves(const FcShape& s, int batch, int slices) {
    const int cols = s.mean_tiles * s.bw, steps = cols * elem_size(s.wdtype) / 64;
    const bool small = batch <= 8 ? steps <= 16 : (s.wdtype == PIVOT_F16 || batch <= 16) && (s.bh == 8 ? steps / 2 : steps) <= 8;   // (of tiles 8 high two sets make a step)
    int nw = small || (s.wdtype == PIVOT_F16 && (long long)s.nchunks * slices >= 512) ? 2 : 4;
    return nw == 2 && s.chunk_tiles > 2 * frag_wave_tiles(s) ? 4 : nw;
}
// Batch rows one launch row covers in the kernel's epilogue and in the workspace (grid.y repeats it).
int fc_batch_tile(const FcShape& s, int batch) {
    if (s.layout != PIVOT_BRC) return 1;     // the column-major kernels take one batch row per launch row
    const int path = fc_path(s, batch);
    if (path == kPathFrag) { int sl, nbt; frag_split(s, batch, &sl, &nbt); return 16 * nbt; }
    if (path == kPathMfmaLds) return mfma_lds_rows(batch);
    if (path == kPathMfmaXrow) return 16;
    return batch >= 3 ? 4 : batch;
}

// Largest number of row slices <= want that the chosen kernel supports: a
// slice of the vector kernel has at least 8 rows and is a whole number of 1 KB
// wave-loads or a whole fraction of one (a wave-load then takes the same rows
// of several consecutive tiles), a slice of the matrix kernel whole MFMA row blocks.
int fc_row_slices(const FcShape& s, int batch, int want) {
    const int layout = s.layout, wdtype = s.wdtype, bh = s.bh, bw = s.bw;
    if (layout != PIVOT_BRC) return 1;       // a row slice is contiguous only in row-major tiles
    if (fc_path(s, batch) == kPathFrag) { int fs, nbt; frag_split(s, batch, &fs, &nbt); return fs; }
    int sl = want < 1 ? 1 : want;
    // The LDS-fed matrix-core kernel beyond 8 batch rows (several launch rows of 8): every row slice of a block
    // row stages the same x-segments again, so at most two slices (4096x4096, 64x16 tiles, cold, four slices ->
    // two: 10 % kept, batch 12 / 16 / 24 / 32 / 64: 5.9 -> 5.4, 5.9 -> 5.4, 7.2 -> 6.4, 8.45 -> 7.1, 12.8 -> 10.3
    // us; 25 % kept, batch 24 / 32: 10.8 -> 9.3, 12.7 -> 10.2; one slice: 6.6 at batch 16; up to batch 8 four
    // slices are the faster, 4.9 against 5.3 us).
    if (sl > 2 && batch > 8 && fc_path(s, batch) == kPathMfmaLds) sl = 2;
    if (fc_path(s, batch) != kPathVector) return mfma_slices(s, sl);
    const int vec = 16 / elem_size(wdtype), rpw = 64 / (bw / vec > 0 ? bw / vec : 1);
    while (sl > 1) {
        const int bhs = bh / sl;
        if (bh % sl == 0 && bhs >= 8 && (bhs % rpw == 0 || rpw % bhs == 0)) break;
        sl /= 2;
    }
    return sl;
}

// Arrival counters of split block rows: one 256-byte line per (launch row, block row, row slice).  Plans without split
// block rows use none.
size_t run_ticket_bytes(const HostPlan& hp, int batch, int x_from) {
    if (hp.max_parts <= 1) return 0;
    size_t most = 0;
    for (int x_vec : {0, 1}) {                       // whatever rows of x the run brings
        FcShape s = fc_shape(hp, x_from);
        s.x_vec = x_vec;
        const int nbt = fc_batch_tile(s, batch), launch_rows = (batch + nbt - 1) / nbt;
        most = std::max(most, (size_t)4 * kTicketStride * hp.nbr * launch_rows * fc_row_slices(s, batch, hp.row_slices));
    }
    return most;
}

// The counter region of a workspace is sized for the largest number of launch rows any batch up to 64 can have, so
// that its size, and with it the place of everything that follows it, does not depend on the batch of a run: counters
// are only ever touched as counters (every run leaves them at zero), never overlaid by another batch's partial sums.
// kXNoCopy, which only runs with the built-in scratch take, counts where the vector kernel is all there is beside the
// form with the copy; fp16 tiles of an MFMA shape have forms of 8 and 16 rows, and the vector kernel, with up to 16
// launch rows, only stands in for them where the copy does not fit (counted there, by run_ticket_bytes).
size_t count_ticket_bytes(const HostPlan& hp) {
    size_t most = 0;
    for (int x_from : {kXNoCopy, kXNatural, kXBlock}) {
        if (x_from == kXNoCopy && mfma_kind(hp.d.wdtype, hp.d.bh, hp.d.bw) >= 0) continue;
        for (int batch = 1; batch <= 64; ++batch) most = std::max(most, run_ticket_bytes(hp, batch, x_from));
    }
    return most;
}

// (For rows of x that are whole aligned vectors where K is: other rows take launch rows of 8 batch rows instead of 16,
// which need no more.)
size_t fc_partial_bytes(const HostPlan& hp, int batch, int x_from) {
    if (hp.max_parts <= 1) return 0;
    const int nbt = fc_batch_tile(fc_shape(hp, x_from), batch);
    const int ngy = (batch + nbt - 1) / nbt;
    return align_up((size_t)4 * hp.nchunks * hp.d.bh * nbt * ngy, 256);
}

size_t fc_gather_bytes(const HostPlan& hp, int batch) {
    if (!fc_wants_frag(fc_shape(hp, kXNatural), batch)) return 0;
    return align_up((size_t)batch * hp.K_pad * elem_size(hp.d.wdtype), 256);
}

// "pivot::<kernel and template arguments>" as a profiler prints it
template <typename... A>
static std::string kernel_name(const char* fmt, A... args) {
    char buf[160];
    snprintf(buf, sizeof buf, fmt, args...);
    return std::string("pivot::") + buf;
}

int launch_fc(const FcLaunch& L, std::string* describe) {
    const int xlen = L.x_block_order ? L.K_pad : L.K;
    const bool vec_rows = xlen % (16 / elem_size(L.wdtype)) == 0 && L.ldx == xlen && (reinterpret_cast<uintptr_t>(L.x) & 15) == 0;
    const FcShape shape{L.layout, L.wdtype, L.bh, L.bw, L.lds_tiles, L.chunk_tiles, L.xrow_len, mean_tiles_of(L.T, L.nchunks), L.nchunks, L.x_from, L.row_slices, vec_rows};
    const int path = fc_path(shape, L.batch);
    const bool ml = path == kPathMfmaLds, mx = path == kPathMfmaXrow;
    const int nbt = fc_batch_tile(shape, L.batch);
    const int ngy = (L.batch + nbt - 1) / nbt;
    const int sl = fc_row_slices(shape, L.batch, L.row_slices);
    const int bhs = L.bh / sl;
    int nw = (L.wg_waves == 16 || L.wg_waves == 8) ? L.wg_waves : 4;
    // one wavefront per work item: the vector kernel at batch 1 with the gather from global memory (tiny layers)
    const bool one_wave = L.wg_waves == 1 && L.layout == PIVOT_BRC && path == kPathVector && nbt == 1;
    if (one_wave) nw = 1;
    if (ml && nw > 8) nw = 8;                // the LDS-fed matrix-core kernel comes with 4 or 8 wavefronts
    const int es = elem_size(L.wdtype);

    FcArgs a;
    a.vals = L.vals; a.xidx = L.xidx; a.chunks = reinterpret_cast<const int4*>(L.chunks);
    a.bias_p = L.bias_p; a.scatter = L.scatter;
    a.x = L.x; a.y = L.y; a.partials = L.partials; a.tickets = L.tickets;
    a.ldx = L.ldx; a.ldy = L.ldy; a.batch = L.batch; a.act = L.act;
    a.nchunks = L.nchunks; a.nbr = L.nbr;
    a.out_form = (L.out_f16 ? kOutF16 : 0) | (L.out_frag ? kOutFrag : 0); a.out_pad = L.out_frag ? L.out_pad : 0;
    a.slices = sl; a.bh_full = L.bh; a.xn_vecs = 0;
    a.uniform_ct = L.uniform_ct; a.uniform_parts = L.uniform_parts;
    a.T = L.T; a.chunk_tiles = L.chunk_tiles;
    a.trace = nullptr;
#ifdef PIVOT_TRACE
    // timeline builds: where the vector kernel puts its time stamps (8 x int64 per wavefront of the launch)
    if (const char* e = getenv("PIVOT_TRACE_PTR")) a.trace = reinterpret_cast<long long*>(strtoull(e, nullptr, 0));
#endif
    dim3 grid(L.nchunks, ngy, sl);
    hipStream_t st = reinterpret_cast<hipStream_t>(L.stream);

    if (L.uniform_ct > 0xFFFF || L.uniform_parts > 0x7FFF) a.uniform_ct = a.uniform_parts = 0;   // packed into 16 bits each: fall back to loaded descriptors
    if (path == kPathFrag) {
        if (!L.x_block_order) { set_error("internal: the batched matrix-core kernel needs x in fragment order"); return PIVOT_E_UNSUPPORTED; }
        if (L.bh > 64 || L.batch > 64) { set_error("shape outside the kernel's packed arguments"); return PIVOT_E_UNSUPPORTED; }
        a.xidx = L.col_idx;
        const int fnw = frag_waves(shape, L.batch, sl);
        if (describe) { *describe = kernel_name("fc_frag_kernel<%s, %d, %d, %d, %d>", L.wdtype == PIVOT_F32 ? "float" : "_Float16", bhs, L.bw, nbt / 16, fnw); return PIVOT_OK; }
        using Launch = int (*)(const FcArgs&, int, int, int, dim3, hipStream_t);
        static const Launch by_height[2][3] = {{launch_frag_f32_8, launch_frag_f32_16, launch_frag_f32_32},
                                               {launch_frag_f16_8, launch_frag_f16_16, launch_frag_f16_32}};
        return by_height[L.wdtype == PIVOT_F32 ? 0 : 1][bhs == 8 ? 0 : (bhs == 16 ? 1 : 2)](a, L.bw, nbt / 16, fnw, grid, st);
    }
    if (mx) {
        if (L.chunk_tiles > 0xFFFF || L.bh > 64) { set_error("shape outside the kernel's packed arguments"); return PIVOT_E_UNSUPPORTED; }
        int kind = mfma_kind(L.wdtype, L.bh, L.bw);
        if (kind == 1 && L.bw == 16 && bhs % 32 != 0) kind = 2;
        // rows that are not whole aligned vectors, densely packed, start anywhere in their first piece of 16 bytes
        const int vecs = vec_rows ? xlen / 8 : (xlen + 7 + 7) / 8;
        a.xn_vecs = xrow_pack(vecs, vecs * 8 - xlen, L.ldx == xlen, vec_rows);
        const size_t steps_cols = ((size_t)(a.uniform_ct > 0 ? a.uniform_ct : L.chunk_tiles) + 1) * L.bw;
        size_t smem = (size_t)16 * xrow_bytes(vecs) + steps_cols * 4;
        const size_t red_bytes = (size_t)8 * bhs * 16 * 4;
        smem = align_up(smem > red_bytes ? smem : red_bytes, 16);
        if (vecs > 513 || steps_cols > 8192 || smem > 158 * 1024) { set_error("internal: x does not fit the LDS copy (%zu bytes)", smem); return PIVOT_E_UNSUPPORTED; }
        if (describe) { *describe = kernel_name("fc_mfma_xrow_kernel<%d, %d, %d, %d>", kind, bhs, L.bw, xrow_xv(a.xn_vecs)); return PIVOT_OK; }
        return launch_mfma_xrow_f16(a, kind, bhs, L.bw, grid, smem, st);
    }
    // staged x: nbt rows of (tiles per chunk)*bw elements, plus 16 bytes whose last element is the dump slot
    // (the kernels derive the same stride from their preloaded arguments)
    // the LDS-fed matrix-core kernel takes slices that are not whole 32-row blocks of 16-column tiles as pairs
    // of tiles (16x16x32 MFMA) and keeps 16 zeroed columns after the last staged tile
    int kind = mfma_kind(L.wdtype, L.bh, L.bw);
    if (ml && kind == 1 && L.bw == 16 && bhs % 32 != 0) kind = 2;
    const int xs_stride = (a.uniform_ct > 0 ? a.uniform_ct : L.chunk_tiles) * L.bw + (ml && kind == 2 ? 16 : 0) + 16 / es;
    size_t xs_bytes = (size_t)nbt * xs_stride * es;
    size_t red_bytes = (size_t)nw * bhs * nbt * 4;
    // x-resident variant: every work item first copies the whole of x (nbt rows) into LDS with independent
    // coalesced loads and gathers from there.  Taken when the rows are 16-byte vectors (densely packed if there
    // is more than one: the kernel then derives the row stride from its preloaded arguments), a thread has to hold at
    // most 8 of them, everything fits in 64 KB of LDS, and the work item streams at least 32 KB of weights
    // (measured at batch 1, where the global form needs no barrier at all because every wavefront stages for
    // itself: below that the copy and its barrier cost 0.3 us warm and gain nothing cold, 1024x1024 fp32 3.19
    // either way, 4096x4096 fp32 at 10 % 4.02 / 4.03; at 40 KB they gain 0.2 us cold, 4096x4096 fp16 at 25 %
    // 4.75 -> 4.54; at 58 KB 0.3 us, 4096x9216 fp32 5.63 -> 5.27; dense 4096x4096 fp16 0.2 us).  With several batch rows the gather issues a load per element and
    // row, so there the copy is also taken as soon as it needs no more loads than the gather would
    // (4096x4096 fp16 at 10 % kept: batch 2 4.16 -> 4.02 us cold, batch 4 4.75 -> 4.43; at 25 %, batch 2:
    // 5.49 -> 4.98; at 5 %, where the gather is the shorter, the copy was 0.1 us slower; warm launches pay
    // 0.2-0.4 us for it).
    if (L.chunk_tiles > 0xFFFF || L.bh > 64 || L.batch > 64) { set_error("shape outside the vector kernel's packed arguments"); return PIVOT_E_UNSUPPORTED; }
    const int vec = 16 / es;
    int xres = 0;
    size_t xn_bytes = 0;
    const size_t item_bytes = (size_t)(a.uniform_ct > 0 ? a.uniform_ct : L.chunk_tiles) * bhs * L.bw * es;
    const size_t staged_cols = (size_t)(a.uniform_ct > 0 ? a.uniform_ct : L.chunk_tiles) * L.bw;
    if (L.layout == PIVOT_BRC && L.x_resident != 0 && !one_wave &&
        (L.x_resident == 2 || item_bytes >= 32 * 1024 || (nbt >= 2 && staged_cols * vec >= (size_t)xlen)) && xlen % vec == 0 && (nbt == 1 || L.ldx == xlen) &&
        (reinterpret_cast<uintptr_t>(L.x) & 15) == 0) {
        const size_t vectors = (size_t)nbt * (xlen / vec);
        xn_bytes = (size_t)nbt * xlen * es + 16;
        if (vectors <= (size_t)8 * nw * 64 && xn_bytes + xs_bytes <= 64 * 1024 && red_bytes <= 64 * 1024) {
            // form 1 (everything requested in one burst) for regular schedules whose work item is in flight whole
            // with the first loads (8 KB per wavefront); form 2 (x stored to LDS between the two halves of the
            // first weight loads) for irregular schedules and for longer work items, whose refills then start sooner
            xres = (a.uniform_ct > 0 && item_bytes <= (size_t)nw * 8 * 1024) ? 1 : 2;
        } else if (!ml && nbt == 1 && vectors <= (size_t)16 * 8 * 64 && xn_bytes + xs_bytes <= 144 * 1024 &&
                   (size_t)L.nchunks * sl <= (size_t)device_cus() &&
                   (L.x_resident == 2 || (size_t)(a.uniform_ct > 0 ? a.uniform_ct : L.chunk_tiles) * L.bw * 128 >= 2 * xn_bytes)) {
            // Long x (beyond 64 KB of LDS or 8 vectors per thread): 8 wavefronts hold up to 16 vectors each and
            // the workgroup takes most of the 160 KB of a compute unit, so this form is only used when every
            // work item still gets a compute unit of its own.  It replaces a gather that moves a whole cache
            // line per element by a copy that moves every line once (25088 inputs, 78 tiles per work item:
            // 320 KB of lines per work item against 100 KB), so it is taken only when the gathered lines are at
            // least twice the copy (16384 inputs, 8 tiles of 64 columns per work item: 64 KB either way, and the
            // copy was measured 0.6 us slower).
            xres = 3;
            nw = 8;
            red_bytes = (size_t)nw * bhs * nbt * 4;
        }
    }
    a.xn_vecs = xres ? xlen / vec : 0;
    size_t smem = xres ? xn_bytes + xs_bytes : xs_bytes;
    smem = align_up(smem > red_bytes ? smem : red_bytes, 16);
    if (smem > (size_t)(xres == 3 ? 150 : 64) * 1024) { set_error("chunk does not fit in LDS (%zu bytes)", smem); return PIVOT_E_UNSUPPORTED; }
    if (describe) {
        // the instantiation the per-path launchers pick for these values (they take 8 wavefronts for 16 where
        // they have no 16-wavefront form, and know one LDS-copy form where the vector kernel knows three)
        const char* wt = L.wdtype == PIVOT_F32 ? "float" : "_Float16";
        if (L.layout != PIVOT_BRC) *describe = kernel_name("fc_colmajor_kernel<%s, %d, %d, %d, %d>", wt, L.layout, L.bh, L.bw, nw >= 8 ? 8 : 4);
        else if (ml) *describe = kernel_name("fc_mfma_lds_kernel<%d, %d, %d, %d, %d, %d>", kind, bhs, L.bw, nbt, nw >= 8 ? 8 : 4, xres ? 2 : 0);
        else *describe = kernel_name("fc_gemv_kernel<%s, %d, %d, %d, %d, %d>", wt, bhs, L.bw, nbt, nw, xres);
        return PIVOT_OK;
    }
#if PIVOT_ABLATE & 32
    // ablation build without permutations: batch 1 through the vector kernel only, which then reads the tile
    // list's block columns where it otherwise reads the per-column gather index
    if (L.layout != PIVOT_BRC || ml || nbt != 1) { set_error("this ablation build runs BRC plans at batch 1 only"); return PIVOT_E_UNSUPPORTED; }
    a.xidx = L.col_idx;
#endif
    if (L.layout != PIVOT_BRC) return launch_colmajor(a, L.layout, L.wdtype, L.bh, L.bw, nw, grid, smem, st);
    if (ml) {
        if (!L.xsort) { set_error("internal: the LDS-fed matrix-core kernel needs the packed gather lists"); return PIVOT_E_UNSUPPORTED; }
        a.xidx = L.xsort;
    }
    if (ml) return launch_mfma_lds_f16(a, kind, bhs, L.bw, nbt, nw, xres, grid, smem, st);
    if (L.out_frag) return (L.wdtype == PIVOT_F32 ? launch_gemv_f32_chain : launch_gemv_f16_chain)(a, bhs, L.bw, nbt, nw, xres, grid, smem, st);
    if (L.wdtype == PIVOT_F32) return launch_gemv_f32(a, bhs, L.bw, nbt, nw, xres, grid, smem, st);
    return launch_gemv_f16(a, bhs, L.bw, nbt, nw, xres, grid, smem, st);
}

}  // namespace pivot
