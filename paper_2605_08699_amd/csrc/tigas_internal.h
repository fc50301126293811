// Internal structures shared by the HIP kernels and the host side of libtigas.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

namespace tigas {

constexpr int K1_THREADS = 256;       // one Gaussian per thread in preprocess / duplicate
constexpr int SORT_THREADS = 256;     // 4 wave64 per sort workgroup
constexpr int SORT_CHUNK = 2048;      // keys ranked per workgroup step (4 waves x 8 rounds x 64)
constexpr int SORT_MAX_BLOCKS = 4096; // workgroups per sort pass (at most)
// Chunked scans of per-block counts: one count per thread, so that many short
// workgroups (on many compute units) read in parallel the counts that the
// previous kernel's workgroups on every XCD just wrote.
constexpr int SCAN_THREADS = 256;
constexpr int SCAN_ITEMS = 1;
constexpr int SCAN_CHUNK = SCAN_THREADS * SCAN_ITEMS;  // counts per workgroup of the chunked scans
constexpr int MAX_SORT_PASSES = 8;
// Bucketed depth sort: buckets per view (one per BUCKET_RECORDS records, a
// power of two), the samples that place their boundaries, the bins of the
// samples' distribution, and the elements a workgroup sorts at once.
constexpr int BUCKET_RECORDS = 1024;
constexpr int BUCKET_MAX = 4096;
// Records per segment at most.  The segments that run together on an XCD write
// to the same buckets, and the shorter they are the more of a line they fill
// while it is in the L2: the scatter of 32 views of 3M records takes 880 / 818 /
// 734 / 737 us with 65536 / 32768 / 16384 / 8192, the counting 209 / 209 / 226 / 264.
constexpr int SEG_MAX = 16384;
constexpr int BUCKET_SAMPLES = 16384;
constexpr int BUCKET_BINS = 2048;
constexpr int BUCKET_CDF_WORDS = BUCKET_BINS + 8;  // cumulative counts, smallest and largest sample, shift, scale
constexpr int BUCKET_SORT_CAP = 4096;
// A bucket with more than CROWD_SHARES times its share of a view's records (and
// over BUCKET_SORT_CAP) is crowded: the frame is rendered again with the buckets of
// views that have one parted by order statistics, from SPLIT_SHARES of the samples
// on (fewer, as samples scatter).  Where there is no second attempt, the samples
// tell from CROWD_SHARES on.  200k Gaussians at 960x540, 5500 / 7000 / 12000 of them at one
// depth (3.5, 4.5 and 7.7 shares of 1564): 197 / 224 / 281 us a frame by depth
// ranges, about 163 / 152 / 152 by order statistics, which cost 12 us to form; 150k over
// 40 depths (3.2 shares of 1172 each, which a workgroup sorts fast) 124 and 147.
constexpr uint32_t CROWD_SHARES = 4, SPLIT_SHARES = 2;
constexpr int COL_CHUNK = 32;  // columns per workgroup of a column scan
// A list is divided into at most 2^cells x 2^cells cells of whole 8x8 blocks (cells 2
// or 1; 0: none): log2 of a cell's side for that of the list's.  An entry's word
// holds the cells that its pixel box meets, as a mask of columns and one of rows,
// above the record's number in its view (in cell_rec_bits bits, 24 or 28), so a
// block of the blend tells from the word whether to fetch the record.
constexpr __host__ __device__ int cell_rec_bits(int cells) { return 32 - 4 * cells; }
constexpr __host__ __device__ int cell_log(int list_log, int cells) {
    return list_log - cells < 3 ? 3 : list_log - cells;
}
// Tile placement: cells of the tile grid per workgroup, the units of the depth
// order per view and at most in all, their smallest cost, a Gaussian's cost
// besides its entries, tiles per workgroup of the ranges.
constexpr int COUNT_LISTS_MAX = 8192;  // lists of a view that are placed by counting although no tiles share them
constexpr int TILE_CELLS = 1024;
constexpr int TILE_UNITS = 1536;
constexpr int TILE_UNITS_MAX = 49152;
constexpr int TILE_UNIT_MIN = 4096;
constexpr int TILE_BASE_COST = 8;
constexpr int TILE_FRONT_TILES = 2048;
constexpr int TILE_CHUNK = 16;  // tiles per workgroup of the scan of their counts

// Resident scene (device pointers).  Layout by storage precision:
//   mean:  f32 planes [3][n] (x, y, z)
//   F32:   attr float4 [2][n]: (qw, qx, qy, qz), (ls0, ls1, ls2, logit)
//          sh   float4 [12][n]: 48 floats per Gaussian, coefficient-major (k*3 + ch)
//   F16/BF16: attr uint4 [n]: 8 halves (qw, qx, qy, qz, ls0, ls1, ls2, logit)
//          sh   uint4 [6][n]: 48 halves per Gaussian, coefficient-major
struct SceneView {
    int64_t n;
    int storage;  // 0 f32, 1 f16, 2 bf16
    int sh_degree;
    const float* mean;
    const void* attr;
    const void* sh;  // per Gaussian: sh_stride contiguous 16-byte words (4 floats or 8 halves)
    int sh_stride;
};

// Per-view camera and tiling parameters, computed on the host in FP64 and
// rounded once to FP32.
struct ViewParams {
    float V[9];        // world -> camera rotation R^T, row-major
    float cam[3];      // camera centre t
    float tz_key;      // float((-R^T t)_z): constant term of the FP32 depth key
    float fx, fy, cx, cy;
    float lim_x, lim_y;  // Jacobian clamp: 1.3 x the half-FoV tangents
    int width, height;
    // Tile lists: 2^lx x 2^ly tiles of 2^tw_log x 2^th_log pixels share one
    // (a single tile unless the placement is by counting); tiles_x, tiles_y
    // and tile_base number the lists.  Where the lists are built, a list is what
    // is called a tile.
    int tw_log, th_log, lx, ly, tiles_x, tiles_y;
    int cells;           // log2 of a list's cells a side; the records' list rectangles carry their end cells
    uint32_t tile_base;
    int sh_degree;
    int fmt;             // 0 RGB8, 1 RGBF32
    float bg[3];
    uint64_t out_ptr;    // device address of this view's frame
    SceneView scene;     // the scene this view renders
    // bucketed depth sort: the view's records, its segments of them, its
    // buckets (numbered from a multiple of COL_CHUNK) and the words of its
    // (segment x bucket) counts before them
    uint32_t rec_base, n_pad;
    uint32_t seg_base, nseg;
    uint32_t bkt_base, nbkt;
    uint64_t row_base;
    uint32_t tchunk_base;  // tile placement: chunks of TILE_CHUNK tiles of the views before
};

// Why a frame has to be rendered again: more entries than the buffers hold; depth
// keys that span too much, or crowd in one bucket (only where the caller asked).
constexpr uint32_t FLAG_FULL = 1, FLAG_WIDE = 2, FLAG_CROWDED = 4;
struct FrameCounters {  // as the caller sees them
    uint32_t D;         // duplicates (clamped to 2^32-1)
    uint32_t visible;
    uint32_t fallbacks;
    uint32_t overflow;  // FLAG_*: nothing was emitted
    uint32_t fb_list;   // append cursor of the FP64-fallback list (cleared once counted)
    uint32_t fb_listed; // entries in the FP64-fallback list this frame
};
// On the device D counts list entries, fewer than the (Gaussian, tile) pairs
// where tiles share a list.
struct Counters : FrameCounters {
    uint32_t pairs;
    uint32_t pad;
};

// Preprocess outputs, one slot per record (record = view-local index of a
// Gaussian, padded per view to a multiple of 256).
// One projected Gaussian (record), 64 bytes: all that the blend gathers for
// a list entry lies in one 64-byte segment.
struct alignas(64) Rec {
    float4 r0;   // u_hi, v_hi, u_lo, v_lo
    float4 r1;   // A, B, C, L: alpha = 2^(A dx^2 + B dx dy + C dy^2 + L)
    float4 r2;   // r, g, b, opacity
    uint2 bbox;  // inclusive pixel box: x0 | y0 << 16, x1 | y1 << 16
    uint2 pad;
};
static_assert(sizeof(Rec) == 64, "record is one 64-byte segment");

struct PreOut {
    Rec* rec;           // records (written only for Gaussians that touch a tile)
    uint2* rect;        // per record: tile rectangle tx0 | ty0 << 16, nx | ny << 16 (0 when no tile;
                        // a record is visible when nx ny > 0)
    uint2* srect;       // the visible records' tile rectangles in depth order (last depth pass)
    uint32_t* zkey;     // FP32 depth-key bits
    uint32_t* blk_sum;  // per 256-record block: tile lists touched
    uint32_t* blk_vis;  // per block: records that touch a tile
    uint32_t* blk_fb;   // per block: FP64 fallbacks
    uint32_t* blk_tiles;  // per block: tiles touched (blk_sum: their lists)
    uint32_t* blk_view; // per block: view index
    unsigned long long* vmask;  // per 64 records: which touch a tile
    uint32_t* sample;           // per 64 records: the depth key of one that does (all ones: none)
    uint32_t* chunk_vis;            // per SCAN_CHUNK block counts: visible records,
    unsigned long long* chunk_dup;  // duplicates,
    uint32_t* chunk_fb;             // FP64 fallbacks,
    uint32_t* chunk_dups;           // and (later) depth-ordered duplicate counts
    uint2* fb_list;     // (record, Gaussian) pairs whose conic is recomputed in FP64
    uint32_t fb_cap;
    Counters* cnt;
};

// Double-buffered (key, value, extra) words of a radix sort.
struct SortBuffers {
    uint32_t* key[2];
    uint32_t* val[2];
    uint32_t* ext[2];
    uint32_t* hist;    // [256][segments] digit counts per segment (then each digit's offsets)
    uint32_t* dtot;    // [256] per-digit totals
};

// Per-view totals of the preprocess.
struct ViewCount {
    unsigned long long dups, tiles;  // list entries; (Gaussian, tile) pairs
    uint32_t visible, fallbacks;
    uint32_t start;             // visible records of the views before
    uint32_t ubase, nu, ucost;  // units of the tile placement: of the views before, of this one, cost of one
};

// A segment of a view's records: list entries, (Gaussian, tile) pairs, visible
// records, FP64 fallbacks, smallest and largest visible depth key.
struct SegTotals {
    unsigned long long dups, tiles;
    uint32_t visible, fallbacks, lo, hi;
};

// Scratch of the bucketed depth sort (all views of a launch sequence).
struct BucketMem {
    uint4* elem;         // [visible] (depth key, record, packed rectangle, -) in bucket order
    uint32_t* rows;      // per view [segments][buckets]: counts, then exclusive prefixes over segments
    uint32_t* start_in;  // per bucket: records of the buckets before it in its chunk of COL_CHUNK
    uint32_t* tot;       // per bucket: records
    uint32_t* chunk;     // per chunk of COL_CHUNK buckets: records
    uint32_t* cdf;       // per view: BUCKET_CDF_WORDS
    SegTotals* seg;      // [segments]
    uint32_t* cost;      // per bucket: its entries and TILE_BASE_COST per record,
    unsigned long long* ccost;  // and per chunk (cleared each frame)
    ViewCount* vc;       // per view
};

// Scratch of the tile placement.
struct TileMem {
    uint32_t nunits;      // units aimed at; rows holds one more per view
    uint32_t stride;      // words of a row: the tiles of the largest view
    uint32_t* rows;       // [units][stride]: counts, then exclusive prefixes over a view's units
    uint2* urange;        // per unit: its range of the depth order
    uint32_t* start_in;   // per tile: entries of the tiles before it in its chunk
    uint32_t* tot;        // per tile: entries
    uint32_t* chunk;      // per chunk of TILE_CHUNK tiles: entries
};

// Arrays cleared (as u32 words) by the first kernel after preprocess.
struct ZeroList {
    static constexpr int N = 3;
    uint32_t* p[N];
    uint32_t n[N];
};

struct SortPass {
    int shift;
    int bits;   // <= 8
};

// ---- launchers (kernels.hip) ----
void launch_preprocess(const SceneView& s, const ViewParams* views_dev, const ViewParams* views_host, int nviews,
                       uint32_t rec_base, uint32_t n_pad, uint32_t view_base, const PreOut& o, hipStream_t st);
// One view's parameters stored to device memory by a kernel (argument by
// value), which also clears nclear words (no memset node in captured sequences).
void launch_store_view(const ViewParams& v, ViewParams* dst, uint32_t* clear, uint32_t nclear, hipStream_t st);
void launch_scan_visible(const PreOut& o, int nblk, uint32_t* blk_off, Counters* cnt, uint32_t cap,
                         const ZeroList& zl, hipStream_t st);
// Visible records as (depth key, record) pairs; with ext, also each one's
// tile rectangle packed into one word (views of at most 256 x 256 tiles).
// The same launch recomputes, in FP64, the conic of every Gaussian
// preprocess listed as near-singular (before anything reads it).
void launch_compact(const PreOut& o, int nblk, const uint32_t* blk_off, uint32_t* key, uint32_t* val, uint32_t* ext,
                    const ViewParams* views_dev, hipStream_t st);
// The depth-ordered tile rectangles come packed (sorted_packed, carried by the
// depth passes) or, when that is null, as two words (sorted_rect).
void launch_duplicate(const PreOut& o, int nblk, const uint32_t* sorted_rec, const uint2* sorted_rect,
                      const uint32_t* sorted_packed,
                      uint32_t* blk_sum2, uint32_t* blk_off2, const Counters* cnt, uint32_t cap,
                      const ViewParams* views_dev, uint32_t* tile_out, uint32_t* val_out, uint32_t* depth_out,
                      hipStream_t st);
// Duplicates with tighter tile culling (packed rectangles only): per
// (Gaussian, tile of its rectangle), kept when the Gaussian can reach the
// skip threshold at one of the tile's pixels; the kept entries in emission
// order (blk_cnt, blk_off: per-256-Gaussian kept counts and their scan), and
// the kept count stored as the frame's D.
void launch_duplicate_culled(const PreOut& o, int nblk, const uint32_t* sorted_rec, const uint32_t* sorted_packed,
                             uint32_t* blk_cnt, uint32_t* blk_off, Counters* cnt, const ViewParams* views_dev,
                             int tile_w, int tile_h, uint32_t* tile_out, uint32_t* val_out, uint32_t* depth_out,
                             hipStream_t st);
// Bucketed depth sort of every view's visible records: val / ext receive the
// record ids (in a view with cells, the record's number in it and its rectangle's
// end cells) and packed list rectangles view by view in depth order, equal
// depths in record order (views of at most 256 x 256 tiles).  The same
// launches set the frame's counters, clear zl and recompute, in FP64, the
// conic of every Gaussian preprocess listed as near-singular.  flag_wide: a
// frame whose depth keys span 2^27 or more is flagged and left unsorted (the
// caller renders it again with the four-pass radix sort); flag_crowd: so is one with
// a crowded bucket (the caller renders it again with split).  split (0: off): views
// with more than this many shares of the samples in a bucket are parted so that
// no bucket is long.
// seg_len: records per segment; nseg, nchunks: segments and bucket chunks of
// all views; nunits: of the tile placement that follows.
void launch_bucket_sort(const PreOut& o, const BucketMem& b, const ViewParams* views_dev, int nviews, uint32_t nseg,
                        uint32_t nchunks, uint32_t seg_len, Counters* cnt, uint32_t cap, const ZeroList& zl,
                        bool flag_wide, bool flag_crowd, uint32_t split, uint32_t nunits, uint32_t* val, uint32_t* ext,
                        hipStream_t st);
// Runs LSD passes over the count selected by `which` (0 duplicates, 1 visible)
// starting in buffer `start`; returns the buffer index holding the result.
// With `rect_src`, the last pass also writes rect_src[value] to rect_dst in
// sorted order.
int launch_sort(const SortBuffers& b, const SortPass* passes, int npasses, int which, uint32_t cap, int nblocks,
                int start, bool extra, Counters* cnt, const uint2* rect_src,
                uint2* rect_dst, hipStream_t st);
// Tile ranges of the sorted list.  host_cnt: pinned host memory (or device
// memory) that receives a copy of the counters.
void launch_ranges(const uint32_t* tile_sorted, const Counters* cnt, uint32_t cap, uint2* ranges, FrameCounters* host_cnt,
                   hipStream_t st);
// The blend's dense-first dispatch order of n_tiles tiles (longest lists
// first) from their ranges: order receives a permutation of 0 .. n_tiles-1.
void launch_tile_order(const uint2* ranges, uint32_t n_tiles, uint32_t* order, hipStream_t st);
// Tile placement by counting (packed rectangles): from the depth-ordered
// records and packed rectangles, writes each (Gaussian, tile) entry's record
// id to its sorted position in val_out (in a view with cells, the record's number
// in it and the cells of the list that the entry covers; with
// tile_out/depth_out, also its tile
// id and depth word), the tile ranges and the counters to host_cnt.  The
// depth order is the bucketed one (view by view, b filled in by
// launch_bucket_sort) or, flat, a single view's from the radix passes.
// nchunks: chunks of TILE_CHUNK tiles over all views.  order (may be null):
// receives the blend's dense-first dispatch order (a single view).
void launch_tiles(const TileMem& m, const BucketMem& b, const ViewParams* views_dev, const ViewParams* views_host,
                  int nviews, uint32_t nrec, const Counters* cnt, bool flat, uint32_t nchunks, const uint32_t* rec,
                  const uint32_t* packed, uint2* ranges, uint32_t* order,
                  FrameCounters* host_cnt, uint32_t* val_out, uint32_t* tile_out, uint32_t* depth_out,
                  const uint32_t* zkey, hipStream_t st);
// Baseline JPEGs of RGB8 frames: one workgroup per restart interval of
// JPEG_SEG_MCUS MCUs, the intervals of up to JPEG_MAX_JOBS frames in one pair
// of launches.
constexpr int JPEG_SEG_MCUS = 40;
constexpr int JPEG_SEG_THREADS = 512;
constexpr int JPEG_PACK_THREADS = 256;
constexpr int JPEG_MAX_JOBS = 16;
// Annex K base tables (Tables K.1, K.2), row-major, and their scaling by
// quality: 5000/q below 50, else 200 - 2q percent, rounded, within 1..255.
#define JPEG_QLUMA                                                                                            \
    {                                                                                                         \
        16, 11, 10, 16, 24, 40, 51, 61, 12, 12, 14, 19, 26, 58, 60, 55, 14, 13, 16, 24, 40, 57, 69, 56, 14,   \
            17, 22, 29, 51, 87, 80, 62, 18, 22, 37, 56, 68, 109, 103, 77, 24, 35, 55, 64, 81, 104, 113, 92,   \
            49, 64, 78, 87, 103, 121, 120, 101, 72, 92, 95, 98, 112, 100, 103, 99                             \
    }
#define JPEG_QCHROMA                                                                                          \
    {                                                                                                         \
        17, 18, 24, 47, 99, 99, 99, 99, 18, 21, 26, 66, 99, 99, 99, 99, 24, 26, 56, 99, 99, 99, 99, 99, 47,   \
            66, 99, 99, 99, 99, 99, 99, 99, 99, 99, 99, 99, 99, 99, 99, 99, 99, 99, 99, 99, 99, 99, 99, 99,   \
            99, 99, 99, 99, 99, 99, 99, 99, 99, 99, 99, 99, 99, 99, 99                                        \
    }
__host__ __device__ constexpr int jpeg_quant_step(int base, int quality) {
    const int s = quality < 50 ? 5000 / quality : 200 - 2 * quality;
    const int q = (base * s + 50) / 100;
    return q < 1 ? 1 : q > 255 ? 255 : q;
}
// Header bytes that differ between frames: the two quantisation tables, then
// height and width (two bytes each).
constexpr uint32_t JPEG_HDR_QLUMA = 25, JPEG_HDR_QCHROMA = 90, JPEG_HDR_SIZE = 159;
struct JpegJobArgs {
    const uint8_t* rgb;  // H x W x 3, row-major
    uint8_t* out;
    uint64_t capacity;
    uint64_t* out_len;   // total length (written by the last interval)
    int width, height, w8, quality;
    uint32_t n_mcu, nseg;  // 8x8 pixel blocks, restart intervals
    uint32_t seg_base;     // intervals of the jobs before this one
};
struct JpegBatch {
    JpegJobArgs job[JPEG_MAX_JOBS];
    int njobs;
    uint32_t seg_words, header_len;
    float dct[64];          // M[k][n] = c(k)/2 cos((2n+1) k pi/16), FP32
    const uint32_t* huff;   // [4][256] length << 16 | code: DC luma, AC luma, DC chroma, AC chroma
    const uint8_t* header;  // header template
    const uint8_t* zigzag;  // row-major index of each scan position
    uint32_t* bits;         // [intervals][seg_words] entropy-coded bits, padded with ones
    uint32_t* seg_bytes;    // [intervals] bytes before stuffing
    uint32_t* seg_len;      // [intervals] output bytes (stuffing and marker included)
};
void launch_jpeg(const JpegBatch& a, uint32_t nseg, hipStream_t st);
// Composites the lists (n_lists of all views; a single view's in `order`).
// cull: drop the entries whose exponent stays below the skip threshold on a
// block's whole pixel block (they would be skipped at every pixel anyway).
void launch_blend(const ViewParams* views_dev, const ViewParams* views_host, int nviews, uint32_t n_lists,
                  const uint2* ranges, const uint32_t* vals, const PreOut& o, uint32_t nrec,
                  unsigned long long* work, bool cull, const uint32_t* order, hipStream_t st);
void launch_wave_scan_selftest(const uint32_t* in, uint32_t* out, int n, hipStream_t st);

// Per-launch timing for profiling: while a timer is installed for the calling
// host thread, every kernel launch is bracketed by two events on its stream
// (never used for captured launches).
struct KernelTimer {
    virtual void before(const void* kernel, hipStream_t st) = 0;  // kernel: its host-side handle
    virtual void after(hipStream_t st) = 0;
    virtual ~KernelTimer() = default;
};
extern thread_local KernelTimer* g_kernel_timer;

// Sets the message tigas_last_error() returns on the calling thread.
void set_last_error(const char* msg);

}  // namespace tigas
