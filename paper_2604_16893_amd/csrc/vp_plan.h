// vp_plan.h -- device-side plan of one vp_preprocess_batch call.
//
// The host planner (vp_api.cpp) validates the items, derives their work units,
// row offsets and the tables not computed on the device, packs everything into
// one blob and has it copied into the caller's workspace on the call's stream;
// the kernels (vp_kernels.hip) read it from there.  Layout of the blob, each
// section aligned to 256 bytes:
//   DevItem    items[n_items]
//   int32      tile_prefix[n_items + 1]   general-kernel work of item b: [prefix[b], prefix[b+1])
//   int32      indices[sum of padded counts]  source frame of every (frame pair, dt)
//   int32      tables[...]                filter tables from the host, 4-byte words: the general
//                                         kernel's and the uint8 writer's
//   StreamUnit units[...]                 streaming-kernel work units
//   uint32     wgs[...]                   streaming-kernel workgroups, grouped per launch:
//                                         unit index | column band << 20, or kNoWork
//   TableJob   jobs[...]                  pieces of the tables that follow
//   int32      tables[...]                the float streaming kernels' tables, computed on the
//                                         device (not part of the copy, but for some plans of
//                                         the no-alloc entry; word offsets from the first tables
//                                         section like the others)
//
// Tables (word offsets into `tables`; items with the same axis share them):
//   window table of an axis n_in -> n_out, K taps:
//       int32 start[n_out]; int32 count[n_out]; float weight[n_out][K]
//     (the streaming kernels, but for the writer's matrix-core form, read a
//     table of the starts alone)
//   slot table of a y axis n_in -> n_out (streaming kernel), M slots:
//       [n_in + 6] rows of M words: float weight[slot]
//         -- output row i is accumulated in slot i mod M from the first row of
//            its window to its close row; weight[s] is 2^24 times the weight
//            of source row y in the output row that has slot s at y, or zero
//            (the kernel reads source bytes as f16 denormals, b * 2^-24)
//       int32 close_row[n_out + 2]   (the last two entries are INT32_MAX: the
//            kernels read one close row ahead, up to entry n_out + 1)
//         -- the row after which output row i is complete, the last row of its
//            window: never decreasing, and several output rows may close on
//            one row (an upscaled axis, the bottom border)
//   fixed-point window table (uint8 writer): as the window table, with int32
//       weights in units of 2^-22
//   column table of an x axis (streaming kernels), KX taps, for output bands
//   of `band` columns whose source pixels fit a row of `row_px` pixels (the
//   y-first kernel's LDS row; the x-first kernel passes W + KX, a bound no
//   window reaches):
//       int32 start[n_out]; float weight[n_out][KX]
//     -- start is relative to the first source pixel of the output's band
//        (the window start of the band's first column) and start + KX never
//        passes row_px; weights are shifted and zero-padded to match.
// The uint8 writer's column, slot and digit tables are described at their
// builders in vp_api.cpp.
#pragma once

#include <cstdint>

#include <hip/hip_runtime_api.h>

namespace vp {

constexpr int kPatch = 16;
constexpr int kWin = 32;              // merge window edge in pixels (patch * merge)
constexpr int kRow = 1536;            // 3 * 2 * 16 * 16
constexpr int kWinElems = 4 * kRow;   // one merge window of one frame pair
constexpr int kGenericThreads = 256;
constexpr int kGenericTCap = 8192;    // floats of the general kernel's LDS column tile
constexpr int kSlotWords = 16;        // most slots of a slot table (x-first kernel)
constexpr int kStreamSlots = 8;       // most slots of the y-first kernel and the uint8 writer's dot products
constexpr int kSlotMax = 6;           // zero rows past a slot table's last source row
constexpr int kStreamLdsBudget = 64 * 1024;   // LDS of one streaming workgroup (one wave)

// LDS of one streaming workgroup.  Patch 16 (one wave): its source row (64 *
// px float4 pixels) and the stage of four output rows (3 channels x 4 rows x
// 64 columns).  Patch 14 (four waves: a pair's two frames over two bands):
// four source rows and the stage of `patches` whole output rows of 1176
// values, the patches of the two bands.
constexpr int stream_wave_bytes(int px, int kx, int elem_bytes, int patch, int patches) {
    return (void)kx, patch == 16 ? 64 * px * 16 + 3 * 4 * 64 * elem_bytes
                                 : 4 * 64 * px * 16 + patches * 6 * patch * patch * elem_bytes;
}

// LDS of one x-first streaming workgroup (one wave of cpl columns per lane):
// the stage of four output rows (its lanes load their source windows from
// memory).  Patch 14: a workgroup's stage of `patches` whole output rows.
constexpr int xfirst_wave_bytes(int elem_bytes, int cpl, int patch, int patches) {
    return patch == 16 ? 3 * 4 * 64 * cpl * elem_bytes : patches * 6 * patch * patch * elem_bytes;
}
constexpr int kXFirstTaps14 = 8;   // patch 14: most column taps of an x-first kernel

// uint8 streaming writer: pixels per lane (a band's source span is at most
// 64 * kRsPx pixels), and the LDS of one workgroup (one wave): its source
// row as three byte planes and the stage of four output rows of up to 64
// RGB pixels.
constexpr int kRsPx = 4;
constexpr int resize_stream_bytes() { return 3 * 64 * kRsPx + 4 * 64 * 3; }
// Normalise + patchify, patch 14 (patchify14_kernel): merge windows per
// workgroup.
constexpr int patch14_windows(int out_bf16) { return out_bf16 ? 3 : 2; }

// The uint8 writer's form with both passes on the matrix cores (launch shape
// kx = kRsMmShape; m = T, the loads per chunk of 16 source rows: 4 T lanes of
// four pixels cover a band's source span, plus kRsMmTwo where a group of 16
// output rows can read more than four chunks, plus kRsMmWide where 16 columns
// read more than 64 source pixels; px = A, the pixels that the windows of 16
// columns start on a multiple of: 16, 8 or 1): output columns per wave, most
// chunks that a group of 16 output rows reads, and its LDS: the chunk's source
// pixels as three planes of 16 rows (16 bytes more than a row's pixels, so
// that eight rows' 16-byte reads meet all banks) and a ring of chunks of
// horizontal sums (16 rows x columns x 3 channels).
constexpr int kRsMmShape = 128;
constexpr int kRsMmTwo = 16;
constexpr int kRsMmWide = 32;
constexpr int kRsMmRing = 8;
constexpr int resize_mm_cols(bool wide) { return wide ? 16 : 32; }
constexpr int resize_mm_plane_row(int t) { return 16 * t + 16; }
constexpr int resize_mm_bytes(int t, int ring, bool wide) {
    return 3 * 16 * resize_mm_plane_row(t) + ring * 3 * resize_mm_cols(wide) * 16;
}

// Kernel an item is routed to.
enum Route : int32_t { kRouteGeneric = 0, kRouteStream = 1, kRoutePatch = 2, kRouteResize = 3 };

// uint8 cache writer (resize_u8_kernel): one workgroup of kRsThreads per tile
// of up to 32 output rows x 64 output columns of one frame; the host picks
// smaller tiles where these LDS budgets require it.
constexpr int kRsThreads = 256;
constexpr int kRsChunk = 4;          // source rows staged per horizontal step (kRsThreads / 64)
constexpr int kRsSrcRow = 2048;      // LDS bytes per staged source row
constexpr int kRsMid = 32768;        // LDS bytes of the horizontal pass's uint8 rows
constexpr int kRsQ = 2048;           // int32 weights of one axis per tile
constexpr int kRsRowsMax = 32;
constexpr int kRsColsMax = 64;

struct DevItem {
    const uint8_t* frames;   // [n_src][H][W][3]
    int64_t frame_bytes;     // H * W * 3
    int64_t row_off;         // first output row of the item
    int32_t H, W, h, w;      // source and target size
    int32_t t, hm, wm;       // frame pairs, merge windows along y and x
    int32_t idx_off;         // first entry of the item in `indices` (2 * t entries)
    int32_t ty_off, tx_off;  // window tables of the y and x axes
    int32_t ky, kx;          // tap stride of those tables
    int32_t rh, cw;          // general kernel: output rows / columns per LDS sub-tile
    int32_t route;
    int32_t band;            // streaming kernels: output columns per wave.  y-first 16, 32, 48 or 64, x-first
                             // 64 or 128 (pairs), both for patch 14 a multiple of 7 from 14 to 63; uint8
                             // writer 16 or 32 (matrix cores), 16 to 64 (dot products)
    int32_t sy_off, sx_off;  // streaming kernel: slot and column tables
    int32_t row_px;          // streaming kernels: the column table's row bound (64 * px; x-first W + kx)
    int32_t patch;           // patch edge P (16 or 14): rows of 6 P^2 values, windows of 2P
};
static_assert(sizeof(DevItem) == 104, "DevItem layout");

// One streaming work unit: output rows [i0, i1) of padded frame position p
// of an item; one workgroup per column band of the unit.  Bit kUnitBoth of
// p_flags: the pair's two frames are the same source frame (an image, or an
// odd count padded with its last index), so the unit writes both temporal
// halves of the rows.  p < 2^30 always: every frame pair owns at least four
// of the batch's at most 2^31 - 1 rows.
struct StreamUnit {
    int32_t item;
    int32_t p_flags;   // p | kUnitBoth if the pair's frames are one
    int32_t i0, i1;    // output rows [i0, i1) of the frame
};
static_assert(sizeof(StreamUnit) == 16, "StreamUnit layout");
constexpr int32_t kUnitBoth = 1 << 30;

struct PlanView {
    const DevItem* items;
    const int32_t* tile_prefix;
    const int32_t* indices;
    const int32_t* tables;
    const StreamUnit* units;
    const uint32_t* wgs;
    int32_t n_items;
    int32_t n_tiles;
};

struct Norm {
    float a[3];   // 1 / (255 * std_c)
    float b[3];   // -mean_c / std_c
    float z[3];   // -255 * mean_c: v = a_c * (R + z_c), the same value in pixel units
};

// Streaming workgroup entries: unit index in the low 20 bits, column band
// (at most kWgBandMax) above; kNoWork marks an empty workgroup.
constexpr uint32_t kWgUnitMask = (1u << 20) - 1;
constexpr int kWgBandShift = 20;
constexpr int kWgBandMax = (1 << (32 - kWgBandShift)) - 2;   // keeps entries below kNoWork
constexpr uint32_t kNoWork = 0xffffffffu;

// One launch of the streaming kernel: workgroups wgs[first, first + count),
// all with the same template shape.  px < 0 marks the x-first kernel:
// xfirst_px(0) one column per lane, xfirst_px(2) column pairs whose second
// window starts at most 2 pixels after the first's.
constexpr int32_t xfirst_px(int db) { return -1 - db; }
constexpr int xfirst_db(int32_t px) { return -1 - px; }
struct StreamLaunch {
    int32_t first, count;
    int32_t m, kx, px;       // accumulator slots, column taps, pixels per lane (or xfirst_px)
    int32_t patch;           // patch edge of the batch (16 or 14)
    int32_t lds_units;       // sizes the LDS: patch 14, most patches of two bands (a workgroup's
                             // columns); uint8 writer's matrix-core form, its ring of chunks
    int64_t cost;            // host only: estimated work (source pixels read)
};

// Fixed device memory for the plan of vp_preprocess_batch_noalloc, one array
// per device (vp_kernels.hip), and its size.  noalloc_plan_memory() gives the
// current device's copy of the array, looked up once per device; it returns
// a hipError_t value.
constexpr int64_t kNoAllocPlanBytes = int64_t(16) << 20;
int noalloc_plan_memory(void** ptr);

// A piece of a table that the device computes from the axis alone, one
// workgroup's share of the table at word `off`:
//   starts: the window starts of kTablePiece outputs from `base`;
//   slots: the weights and close rows of table_outputs(lanes) outputs from
//     `base` in a slot table of a = M slots;
//   zeros: kTablePiece words from `base` of the same table, those that no
//     output row's weight stands in, and the two close rows past the last;
//   columns: the starts and weights of table_outputs(lanes) outputs from
//     `base` in a column table of a = KX taps.
// `lanes` threads work on one output: a power of two, no fewer than its taps
// (columns: than KX), up to the whole workgroup.
enum TableKind : int32_t { kTableStarts = 0, kTableSlots = 1, kTableZeros = 2, kTableColumns = 3 };
struct TableJob {
    int32_t kind_lanes;   // kind | lanes << 8
    int32_t n_in, n_out, a, band, row_px, off, base;
};
static_assert(sizeof(TableJob) == 32, "TableJob layout");
constexpr int kUploadThreads = 256;
constexpr int kTablePiece = 4 * kUploadThreads;
constexpr int table_outputs(int lanes) { return kTablePiece / lanes; }

// Kernel launchers (vp_kernels.hip).  Return a hipError_t value.
// The plan blob, `bytes` (a multiple of 16, both ends 16-byte aligned) from
// host memory the device can read, and the tables of `n_jobs` pieces (`jobs`
// readable by the device: the blob's, in host memory, or with bytes = 0 a copy
// on the device) into `tables`.
int launch_upload(void* dst, const void* src, int64_t bytes, const TableJob* jobs, int n_jobs, int32_t* tables,
                  hipStream_t stream);
int launch_generic(const PlanView& plan, void* out, int out_dtype, const Norm& norm,
                   hipStream_t stream);
int launch_stream(const PlanView& plan, const StreamLaunch& launch, void* out, int out_dtype,
                  const Norm& norm, hipStream_t stream);
// Normalise + patchify of frames already at the target size: one workgroup
// per merge-window row of a frame pair (tile_prefix counts them per item; for
// patch 14 it counts merge windows).
int launch_patchify(const PlanView& plan, void* out, int out_dtype, const Norm& norm, int patch,
                    hipStream_t stream);
// uint8 cache writer over tile_prefix (items with route kRouteResize: rh x cw
// output tiles, tables holding fixed-point weights); out is the byte buffer.
int launch_resize(const PlanView& plan, void* out, hipStream_t stream);
int launch_resize_stream(const PlanView& plan, const StreamLaunch& launch, void* out, hipStream_t stream);
// Shapes (slots, column taps, pixels per lane) the uint8 streaming writer is built for.
bool resize_stream_supported(int m, int kx, int px);
// Position tables: one thread per output row; tile_prefix holds the items'
// row offsets (cu).  vit / llm may be null.
int launch_positions(const PlanView& plan, int32_t* vit, int32_t* llm, int64_t rows,
                     hipStream_t stream);
// Whether a (m, kx, px) shape has a compiled streaming kernel.
bool stream_shape_supported(int m, int kx, int px);
// Whether an (m, kx, pair offset) shape has a compiled x-first kernel.
bool xfirst_shape_supported(int m, int kx, int db, int patch);

}  // namespace vp
