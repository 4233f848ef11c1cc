// Interface of the matrix-core tile kernel for few to some thousand rows (tiles.hip).
#pragma once
#include "common.h"

namespace milora {

// Tiles and parts of the reduction of one launch; a function of the sizes alone, shared by the launch and the sizing of
// the workspace.
enum TileShape { kTiles64 = 0, kTiles128 = 1, kTiles256 = 2 };
struct TilePlan {
  int shape;  // TileShape: 64 x 64 and 128 x 128 (tiles.hip), 256 x 256 (prefill.hip)
  int tilesM, tilesN;
  int S, steps;          // parts of the reduction, stages of 64 k per part
  size_t partial_bytes;  // fp32 partial tiles in the workspace (0 when S == 1)
};
constexpr int kStreamRows = 32;      // rows up to which a packed linear takes the weight-streaming kernel (decode.hip)
constexpr int kMaxSplitUnits = 512;  // tiles x parts of a launch that cuts its reduction
constexpr int kMaxParts = 8;         // of one reduction
// The first bytes of a routed linear's workspace belong to control words: those of the stream kernels (decode.hip), then the
// part counters of the tile kernel, zeroed by the shrink launch in front of it.  Both keep their data behind them, so calls of
// any sizes and either layout can follow one another on one workspace, and the status word can be asked for after either.
constexpr int kStreamCtrlBytes = 16384;
constexpr int kTileCtrlBytes = kMaxSplitUnits * (int)sizeof(int);
constexpr int kTileCtrlOffset = kStreamCtrlBytes - kTileCtrlBytes;

// `small`: the tiles of tiles.hip are a choice up to kTileMaxRows rows (tiles_supported); `large`: the 256 x 256 kernel is one
// (row-major weights, 64 rows or more).  At least one of them.
TilePlan plan_tiles(int64_t M, int d1, int d2, bool small, bool large);
// The most partial_bytes over the plans of all calls of up to these sizes; never less for a larger size.
size_t partial_bytes_bound(int64_t M, int d1, int d2);
bool tiles_supported(int64_t M, int d1, int d2, bool packed, const void* X, const void* W, const void* Y);
// `row_lora` (always there for packed weights): the LoRA term in fp32 row by row.  Null: by the matrix cores, from the look-ups of
// the other arguments; the rows are then all of the call's.
int routed_linear_tiles(const bf16_t* X, int64_t M, int d1, int d2, const int32_t* row_to_req, const bf16_t* W, bool packed,
                        const int2* row_lora, const bf16_t* bias, const AdapterView& ad, int site, const int32_t* tenant_id, const uint8_t* route,
                        int B, const float* t, size_t t_stride, int parts, const TilePlan& pl, int* cnt, float* partial, bf16_t* Y, hipStream_t st);

}  // namespace milora
