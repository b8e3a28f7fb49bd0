// Shared between the host side of libdgc and its kernels: workspace layout,
// kernel argument blocks and launch geometry.  Nothing here is visible through
// the C ABI.
#ifndef DGC_INTERNAL_H_
#define DGC_INTERNAL_H_

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "dgc_band.h"

#include "dgc.h"

namespace dgc {

inline int64_t ceil_div(int64_t a, int64_t b) { return (a + b - 1) / b; }

// ---- launch geometry -------------------------------------------------------
// Streaming pass: one wavefront owns a contiguous run of kWaveTile elements and
// reads it as kStreamUnroll rounds of one float4 per lane (64 lanes x 16 B =
// 1 KiB per round, fully coalesced).
#ifndef DGC_STREAM_UNROLL
#define DGC_STREAM_UNROLL 4
#endif
constexpr int kStreamUnroll = DGC_STREAM_UNROLL;
constexpr int kWaveTile = 64 * 4 * kStreamUnroll;  // elements per wavefront
constexpr int kStreamThreads = 64;                  // one wavefront per workgroup
constexpr int kStreamWaves = kStreamThreads / 64;
// Workgroups of the streaming pass a compute unit holds at a time.  The pass is faster with few
// wavefronts in flight than with the 32 a compute unit could hold (fewer streams for the memory side
// to interleave), so every launch asks for as much LDS as leaves room for this many workgroups in a
// compute unit's 160 KB.  122 M elements, 0.1 %, eight operand sets in one process (mean; they differ by
// where they lie, by up to 30 us): four 399 us, five 393 (379 to 410), six 400; three workgroups of two wavefronts
// 400 (391 to 414), each set slower than with five of one.  25.6 M elements: four 86.0, five 83.7, six 84.1, three
// of two 84.3.
constexpr int kStreamResidentGroups = 5;
constexpr int kStreamGroupsAfterNorm = 12;  // with clipping on: see launch_stream
constexpr size_t kLdsPerComputeUnit = (size_t)160 * 1024;
// Tile table: one int32 per wave tile = index of the tensor that holds the tile's
// first element, with the top bit set when the tile is not wholly inside one
// tensor or is the ragged last tile (such tiles look up every element's tensor).
constexpr uint32_t kTileMixed = 0x80000000u;

// Emit pass: a workgroup takes kEmitTiles consecutive wave tiles of one tensor.
constexpr int kEmitThreads = 256;
constexpr int kEmitElements = 32768;                  // elements per workgroup
constexpr int kEmitTiles = kEmitElements / kWaveTile;
static_assert(kEmitTiles % (kEmitThreads / 64) == 0, "tiles are dealt round-robin to wavefronts");
// Slots: at the densities the method runs at, a tile of 1024 elements holds one or two selected
// elements.  The streaming pass parks up to kSlotsPerTile of them in a record (kSlotsPerTile
// indices, their v', their u', padding) that it writes in place of the tile's mask words, and
// masks u and v itself, so that the emit pass neither decodes mask words nor goes back to u
// and v for such a tile.  One thread of the emit workgroup per slot of its part.
constexpr int kSlotsPerTile = 8;
constexpr int kSlotRecord = 32;  // 32-bit words per tile: the 128 bytes of the tile's 64 mask words
// Per-tile count of the slotted pass: the top bit says that the tile's line holds mask words although
// the tile lies wholly inside one tensor (it selected more elements than a record holds).
constexpr uint32_t kTileCountHasMask = 0x80000000u;
constexpr uint32_t kTileCountMask = 0xFFFFu;
// Where the re-threshold (or the settling of an exact threshold) lowers the count of a tile with a record, the number of elements that the record holds.
constexpr int kTileCountHeldShift = 16;
static_assert(kWaveTile <= (int)kTileCountMask && kSlotsPerTile <= 15, "a count in 16 bits, a record's in four");
static_assert(3 * kSlotsPerTile <= kSlotRecord, "index, v' and u' of every slot");
constexpr int kEmitSlotThreads = 128;  // emit pass over records: two slots per thread
static_assert(kEmitTiles * kSlotsPerTile == 2 * kEmitSlotThreads, "two slots of the workgroup's tiles per emit thread");
constexpr int kRefineThreads = 1024;                  // the re-threshold pass: one workgroup per tensor
constexpr int kRefinePer = 12;
constexpr int kRefineHeld = 8;   // halves of tiles' records whose keys a thread keeps in registers
constexpr int kRefineList = kRefinePer * kRefineThreads;  // selected elements a workgroup lists in LDS

// Receive side: pairs of one payload handled by one workgroup (kFlatPer per thread) and
// tensors whose counts a workgroup stages in LDS at a time.
constexpr int kFlatThreads = 256;
constexpr int kFlatPer = 4;
constexpr int kFlatChunk = kFlatThreads * kFlatPer;
constexpr int kFlatTensors = 1024;
// A sparse clear has a workgroup at least for every tensor of every payload up to kClearGroups of them (launches
// by tensors against numbered pairs, us: 1000 tensors, sixteen workers 8.8 and 9.5; 4000, four 8.7 and 13.2; 8000, two 10.0
// and 20.0), as many as the longest tensor's pairs ask for up to half as many (500 tensors of 20 M elements, 1 % of
// eight workers: 24.7, with twice as many 29.5, numbered 27.5), and none that would take more than
// kClearRounds chunks one after the other, as where one tensor holds nearly everything.
constexpr int64_t kClearGroups = 16384;
constexpr int64_t kClearRounds = 4;

// Receive side without atomics: a workgroup owns a range of one tensor's elements (a
// whole number of emit workgroups' parts, which follow each other in index order in
// every payload's region), finds the pairs of every payload that fall into it by search,
// and adds them up in LDS.
constexpr int kMergeMaxThreads = 1024;   // 512 threads when there are at most eight payloads
constexpr int kMergeMaxRange = 131072;   // elements per workgroup at most (one bitmap bit each)
constexpr int kMergeEmitBlocks = kMergeMaxRange / kEmitElements;  // emit workgroups' parts per range
// pairs of a range a workgroup takes into registers and its LDS accumulator (512 and 1024 threads);
// a range with more takes a slower way through the same kernel
constexpr int kMergeCapSmall = 4096;
constexpr int kMergeCapLarge = 6144;
static_assert((kMergeMaxRange / 128) % kMergeMaxThreads == 0, "dealt evenly to threads");

// Where the accumulator has a word per element: pairs of a part that a workgroup takes into registers, each with a load and a
// store of its element; with more the whole of the part is read and written.  4096, but 2048 where several payloads spread evenly
// let expect more than 2048: they touch most sectors of a part then, each of them another one with every pair.  By elements and whole
// (accumulating, us): 7 M elements, 1 % of eight workers (2621 pairs a part) 18.4 and 14.2, 256 tensors of 32 K, 2 % of four 16.7 and
// 13.3, but 7.5 % of one 12.9 and 12.7, 64 tensors of 60 K 9.4 and 10.6; and where fewer are expected, pairs that crowd a
// part lie close together in it: 64 of 60 K, 1 % of four (1200), all in an eighth of each tensor 8.4 and 10.9.
constexpr int kDirectPairs = 2048;
constexpr int kDirectPairsMost = 4096;

// Receive side at warm-up densities: a workgroup owns one emit workgroup's part and keeps
// the whole range of the dense vector in LDS.
constexpr int kPartThreads = 1024;
constexpr int kPartChunk = 256;  // slots of a payload a wavefront takes at a time, four consecutive ones to a lane
// Parts times payloads up to which the workgroups of the part kernel, one to a part, search for themselves.  In one
// launch and in two, replacing: 1 M elements (32 parts), four workers, 6.25 %: 10.2 and 11.7 us, sixteen 19.8 and 20.6;
// 7 M (215 parts), four: 13.7 and 15.5, but sixteen 26.4 and 25.4, at 25 % 57.7 and 52.8: without the first guess of the
// searching launch, every wavefront takes five rounds of probes.  And where there is something to search, up to so many lists, none
// of whose first probes another part's search has in the cache already (tensors of 60 K, 6.25 %: 64 of them and eight workers 15.5 and
// 16.0, twelve 20.3 and 19.2, sixteen 24.3 and 22.0; 128 and four 15.0 and 15.9, eight 20.9 and 18.8), and payloads, of
// which a wavefront has two at once from seventeen on and two more one after the other from 33 on (1 M, 24 workers 27.2 and 27.8, 48
// 50.1 and 45.5, 64 64.2 and 57.2; 16 of 60 K, 24 26.8 and 26.6, 32 34.9 and 32.6).
constexpr int64_t kPartSearches = 2048;
constexpr int64_t kPartSearchLists = 512;
constexpr int kPartSearchPayloads = 24;
constexpr int kPartClearThreads = 256;
constexpr int kPartClearLoads = 4;  // loads of four indices a lane has on their way
static_assert(kEmitElements <= 65536 && kEmitElements % kPartThreads == 0 &&
                  (kEmitElements / 32) % kPartClearThreads == 0,
              "dealt evenly");

// Wire format (32-bit values + 16-bit zero-run lengths).  Encoder: pairs handled by one workgroup, the
// lanes of a wavefront on neighbouring pairs.
constexpr int kWireThreads = 256;
constexpr int kWireChunk = 4096;
constexpr int kWireRounds = kWireChunk / kWireThreads;   // rounds of 64 pairs a wavefront takes
// Block sums that the workgroups of the second pass add up for themselves, sixteen rounds of one load of
// four per thread at most; above, a scan launch.  At the limit (67 M pairs) that takes 232 us where the scan
// takes 239 if every region is full, and 44 against 56 if one workgroup in eight has pairs; with 512 of them 13
// against 16.
constexpr int kWireSelfScan = 16384;
// Up to as many workgroup slots the encoder is one launch; their needs lie at the end of the block sums, a word of 64 bits
// each with the call's number above (and a bit that no block sum has).  Calls in two launches and in one, us: in a graph one
// slot 7.1 and 5.3, 64 of 30 pairs 7.3 and 7.0, of 300 10.0 and 8.9, 128 7.4 and 7.5, 10.1 and 9.4, 192 7.4 and 8.4, 10.1 and 10.4, 256 7.4
// and 9.0, 10.1 and 11.2 (every workgroup looks for all the needs before its own); from a stream, where the host enqueues them,
// 128 10.5 and 6.8, 10.8 and 8.6, 256 10.4 and 8.2, 10.6 and 10.3: the line is where calls of that kind stop gaining.  The block
// sums have room for the needs in sets of 24576 elements and more, or of some 500 tensors; in smaller ones the encoder is two launches.
constexpr int kWireOnce = 256;
constexpr uint32_t kWireCall = 0x80000000u;
static_assert(kWireOnce <= kWireThreads, "a thread looks for each slot before its own");
constexpr int kScanThreads = 1024;
constexpr int kScanPer = 8;          // block sums per thread and round of the scan
// Decoder: entries a wavefront decodes at a time (eight per lane: one 16-byte load of runs), positions
// recorded every kDecodeBlock << s entries, s the smallest for which the block sums fit the workspace.
constexpr int kDecodePer = 8;
constexpr int kDecodeBlock = 64 * kDecodePer;
static_assert((kWireChunk >> 3) == kDecodeBlock, "s goes up to 3: the blocks the workspace is sized for");
// Payloads of the direct form that are decoded in one launch: kDecodeGroupsMax workgroups of kDecodeGroup entries at most.
// (Calls in two launches and in one: one payload of 16000 entries 11.0 and 9.6 us, of 32700 11.0 and 10.6, and if it took up to
// 65536 of 45000 10.9 and 11.3; eight payloads 13.3 and 11.0, 18.0 and 16.4, 22.8 and 21.0.)
constexpr int kDecodeGroupThreads = 512;
constexpr int kDecodeGroup = kDecodeGroupThreads * kDecodePer;
constexpr int kDecodeGroupsMax = 8;
// Range form of the decoder: a workgroup owns a range of elements and adds the entries that fall into it
// in LDS, payloads in order (32 KB: four workgroups per compute unit), then touches `dense` once per element.
constexpr int kDecodeRange = 8192;
constexpr int kDecodeThreads = 256;
constexpr int kDecodeTasks = 4;       // blocks of entries a wavefront of the range form holds at a time
constexpr int kDecodeSelfScan = 256;  // block sums a wavefront of the direct form adds up for itself, without a scan launch

// Threshold selection: one workgroup per tensor.
constexpr int kSelectThreads = 1024;
constexpr int kSelectRegKeys = 32;    // candidate keys a thread keeps in registers (32 * 1024 in all)
constexpr int kSelectDirect = 256;    // a bin with at most this many members is ranked directly
constexpr int kSelectBins = 2048;     // 11-bit digits
constexpr int kSelectFloorRounds = 8; // ranks below 16 * this take the short cut over the threads' largest keys
constexpr int kSelectInFlight = 8;    // candidates each thread gathers before using any
// Exact selection (DGC_FLAG_EXACT_SELECT, or a sample as large as the tensor) from more candidates than
// the workgroup's registers hold: select_kernel draws kBandSample elements (blocks of 1 << kBandBlockShift)
// and names a band of keys that holds the wanted rank almost surely, collect_band_kernel reads the
// tensor once, spread over the chip, and lists the keys inside the band, rank_band_kernel ranks them.
// The list of a tensor takes three words per 64 elements of an area of its own.  On the 161-tensor set of
// 25.6 M elements the three kernels take 20 + 55 + 12 us at 0.1 % (the reads, 12 bytes per element, at 5.6 TB/s)
// and no more than 40 us more at 25 %; three workgroup-wide passes over a whole tensor, which are still the way
// out when a band misses, took 1385 us.
// (The sample's blocks are 32 neighbours, so a band misses more often than its seven standard deviations say where
// large values come in clusters: with 2 large rows of 1500 in 3 M elements two calls in a hundred.)
constexpr int kBandSample = kSelectRegKeys * kSelectThreads;
// Bands where the longest such tensor has more than this many elements: up to there the passes of one
// workgroup over it take less than the two launches (one tensor of 33000: 35 against 54 us for the call, 65000:
// 53 and 55, 80000: 60 and 54; 200 of 60000: 117 and 123, of 80000: 153 and 148).  With as many tensors as
// compute units a little earlier (256 of 40000: 102 and 121, of 64000: 159 and 147).
constexpr int64_t kBandFrom = 65536, kBandFromMany = 57344;
constexpr int64_t kBandMany = 256;
// At the lowest densities the band's floor is the threshold of a slotted streaming pass, and refine_kernel finds the
// exact one among what passes and puts the rest back: no pass of its own over g, u, v.
// (The floor lets two to three times as many pass: 4 of a tile's 1024 elements at 0.2 %.  At 0.4 %, where a tile in five
// holds more than a record, 60 tensors of 8 M elements in all take 98 us with bands collected and 108 this way, 12 of 1 M 57 and 71.)
constexpr double kBandInPassDensity = 0.002;
// ... and from a shorter tensor on, because no pass is added (calls at 0.1 %, the passes of one workgroup against this:
// one tensor of 33000 31.2 and 32.0 us, of 50000 39.0 and 32.4, of 65000 46 and 33; 20 of 33000 36 and 44; 100 of 60000
// 75 and 62; one of 50000 with a large row of 100 in the mean of 150 calls, misses and all, 49 and 44).
constexpr int64_t kBandFromInPass = 40960;
// What lies above the floor in the longest tensor, as far as the sample tells, has to fit the list of refine_kernel's
// workgroup, with room for large values that the sample has seen none of.  (A list of 16384: the re-threshold 0.8 us slower.)
constexpr int64_t kBandInPassList = kRefineList * 3 / 4;
// Values that come in rows or runs, or in few magnitudes, are not for a floor (see BandRanks), and which tensors have such
// is known on the device only: a set with tensors so long that a miss would cost a millisecond launches the
// two kernels that collect bands in any case, 7 us where they find nothing to do.  So in such a set the floors
// go into the pass only if the tensors hold more than this in all (calls at 0.1 %, bands collected against this: 6 tensors of
// 1 M 72 and 72 us, 8 of 1 M 82 and 78, 2 of 3.8 M 90 and 95; 12 of 1 M 104 and 92, 8 of 3 M 170 and 146,
// 300 of 70000 190 and 163) ...
constexpr int64_t kBandInPassElements = 8 << 20;
// ... and if some are collected, only if the others hold more than this; otherwise all are.  (4 tensors of 3.8 M, one of
// them with large values in 20 rows, 11.4 M elements in the others: 158 us with their floors in the pass, 150
// without; 161 tensors of 25.6 M, one in fifty with such rows: 158, and 185 without.)
constexpr int64_t kBandMixedElements = 16 << 20;
constexpr int kBandBlockShift = 5;
constexpr int kBandListShift = 6;       // three list words per 64 elements
constexpr int kBandThreads = 256;
constexpr int kBandElements = 8192;     // elements per workgroup of the collecting pass
constexpr int kBandsPerPart = kEmitElements / kBandElements;
struct BandState {  // one per tensor, in a line of its own, because atomics on one line are carried out one
                    // after the other (9 ns each), and 512 bytes from the next (128: the pass 57 instead of 55 us)
  uint32_t floor_key, ceil_key;  // the band: floor_key < key < ceil_key
  uint32_t above, ties, listed;  // keys at or above ceil_key, keys equal to floor_key, keys inside the band
};

// Clipping norm: a fixed number of partial sums keeps the result reproducible.
constexpr int kNormThreads = 256;
constexpr int kNormMaxBlocks = 512;
// The same by workgroups of the selection's launch: shares at most, and how often a workgroup looks for one (a look
// takes about half a microsecond; what is still missing then it sums itself).
constexpr int kNormMaxShares = 128;
constexpr int kNormLooks = 4096;

constexpr int kMaxPayloads = 64;
constexpr size_t kBandStride = 512;
constexpr size_t kPartEntries = 2 * sizeof(int32_t) * kMaxPayloads;  // bytes of a part's entries in the part table
static_assert(sizeof(BandState) <= kBandStride && kBandStride <= kPartEntries, "a tensor with a band has a part at least");
static_assert(kMaxPayloads <= 32768, "a payload's number is packed above a 16-bit index");

// ---- device-resident state (start of the workspace) ------------------------
struct DeviceState {
  double norm;           // L2 norm of g (clipping on)
  float scale;           // factor applied to g
  uint32_t flags;        // DGC_DIAG_*
  uint32_t crowded;      // exact selection in the pass: elements of the tensors whose floor does not go there; zero between calls
  uint32_t wire_call;    // encoder in one launch: number of the next call, and
  uint32_t wire_arrived; // workgroups of this one that have what they need from the others; zero between calls
  uint32_t pad;
};

// Per-tensor selection plan (host arithmetic, uploaded when the density changes).
struct TensorPlan {
  int64_t offset;   // first element of the tensor in the flat buffers
  int64_t n;        // elements
  int32_t count;    // candidates: n (whole tensor) or draws * block
  int32_t rank;     // 0-based descending rank that becomes the threshold
  uint32_t nblocks; // aligned sample blocks in the tensor (sampled mode); by way of a band: its number among such tensors
  int32_t exact;    // 0: sampled; 1: candidates are elements 0..n-1; 2: the same, by way of a band
  int32_t k;             // clamp(ceil(d n), 1, n)
  int32_t refine_limit;  // floor(refine_alpha * k): more passes than this trigger the re-threshold
};

struct WorkspaceLayout {
  size_t state, partials, offsets, out_offsets, plans, thr, tile_info, tile_thr, emit_blocks,
      tile_count, merge_blocks, part_blocks, part_found, wire_first_block, wire_sums, mask,
      total_without_bands,             // what a workspace holds at least
      bands, band_list, total,
      stage_v, stage_u, total_staged;  // staging arrays lie behind `total`: a workspace may end before them
};

// Exact selection with the bands' floors in the streaming pass.
struct FloorArgs {
  int32_t in_pass;        // 0: bands are collected, if there are any
  int32_t* collected;     // device, T: not zero for a tensor whose floor does not go into the pass (the call's counts, which the
                          // emit pass writes last)
  int64_t elements;       // of all tensors with a band
};

struct SelectArgs {
  const float* g;
  const float* u;
  const float* v;
  const TensorPlan* plans;
  DeviceState* state;
  float* thr;
  float* out_thr;       // may be null
  float* tile_thr;      // device, one word per wave tile: the threshold of every tile that lies
                        // wholly inside one tensor; the others hold a NaN put there once by the host
  double* partials;        // partial sums of the squared norm (clipping on)
  int64_t n;               // elements of g
  int32_t looks;           // norm and selection in one launch: how often a workgroup looks for a partial sum (see looks_for)
  double thr_local;        // thr_G / sqrt(N)
  int32_t num_partials;
  float scale_override;    // NaN: unused
  float momentum;
  float scale_const;
  int32_t scale_from_state;  // 1: clipping is on; the scale comes from `partials` and is filed in `state`
  int32_t nesterov;
  int32_t block_shift;  // log2(sample_block)
  BandState* bands;     // device, a slot of kBandStride bytes per tensor that has a band; null: none has
  uint32_t* band_list;  // device, see band_list_begin; null: the set has none
  FloorArgs floor;
  uint32_t seed_lo, seed_hi, iter_lo, iter_hi;
};

struct StreamArgs {
  const float* g;
  float* u;
  float* v;
  uint16_t* mask;              // device, 64 words per wave tile
  const int64_t* offsets;      // device, T + 1
  const float* thr;            // device, T
  const uint32_t* tile_info;   // device, ceil(n / kWaveTile), see kTileMixed
  const float* tile_thr;       // device, ceil(n / kWaveTile), see SelectArgs
  uint32_t* tile_count;        // device, ceil(n / kWaveTile): mask bits set in every tile
  const DeviceState* state;
  int64_t n;
  int32_t num_tensors;
  float momentum;
  float scale_const;
  int32_t scale_from_state;
  int32_t nesterov;
  // staged pass (warm-up densities): selected v' (and u') of every whole tile, masking of u, v in the pass
  float* stage_v;              // device, n floats, or null: plain pass
  float* stage_u;              // device, n floats, or null: no region can overflow, or no factor masking
  int32_t factor_masking;
  int32_t slotted;             // slotted pass (densities up to 0.5 %): records in place of mask words
  FloorArgs floor;             // implies `slotted`
  const TensorPlan* plans;     // device, T: looked at for NaNs with floors in the pass
};

struct EmitBlock {
  int32_t tensor;
  int32_t first_tile;     // first wave tile of the workgroup's run inside that tensor
  int32_t tensor_blocks;  // workgroups that share this tensor
  int32_t pad;
  int64_t lo, hi;         // the tensor's elements [lo, hi): here, so that no workgroup waits for a second table
};

struct RefineArgs {
  const TensorPlan* plans;
  const float* v;              // pre-mask v' as left by the streaming pass
  uint16_t* mask;
  const int64_t* offsets;
  const int64_t* out_offsets;  // payload regions: free until the emit pass, used as scratch
  int32_t* out_idx;
  float* out_val;
  float* thr;
  float* out_thr;              // may be null
  uint32_t* tile_count;        // kept in step with the mask bits the pass clears
  int32_t slotted;             // the streaming pass was a slotted one: records in place of some tiles' mask words
  int32_t factor_masking;
  float* u_out;                // u and v, to put back what is dropped from a record
  float* v_out;
  int32_t on_excess;           // re-threshold tensors that let more than refine_limit pass
  FloorArgs floor;             // settle the threshold of tensors whose floor went into the pass
  const DeviceState* state;
};

struct EmitArgs {
  const EmitBlock* blocks;     // device, one entry per workgroup
  float* u;
  float* v;
  const uint16_t* mask;
  int32_t* out_idx;
  float* out_val;
  const int64_t* offsets;      // device, T + 1
  const int64_t* out_offsets;  // device, T + 1
  int32_t* out_counts;         // device, T
  DeviceState* state;
  int32_t factor_masking;
  const uint32_t* tile_count;  // mask bits per tile, left by the streaming pass
  const float* stage_v;        // as in StreamArgs; null: the streaming pass was a plain one
  const float* stage_u;
  int32_t slotted;             // as in StreamArgs
  const float* settled;        // device, T: the thresholds, where refine_kernel has run on records; else null
  unsigned long long* norm_shares;  // device: cleared for the next call
  int32_t shares;                   // 0: the norm had a launch of its own, or there was none
};

struct MergeBlock {
  int32_t begin;    // first element (flat index) of the range
  int32_t end;      // one past its last element; the range lies inside one tensor
  int32_t tensor;
  int32_t lo, hi;   // the tensor's elements [lo, hi): where in a region a search starts
  int32_t pad;
};

struct PairPayloads {
  const int32_t* idx[kMaxPayloads];
  const float* val[kMaxPayloads];
  int64_t count[kMaxPayloads];
};

struct RegionPayloads {
  const int32_t* idx[kMaxPayloads];
  const float* val[kMaxPayloads];
  const int32_t* counts[kMaxPayloads];
};

// Encoder: regions in, entries out.
struct EncodeArgs {
  const int32_t* idx;            // region layout, ascending inside every region
  const float* val;
  const int32_t* counts;         // device, T
  const int64_t* out_offsets;    // device, T + 1
  const uint32_t* first_block;   // device, T + 1: first workgroup slot of every tensor
  uint32_t* sums;                // device, one word per workgroup slot
  uint16_t* runs;
  float* vals;
  int32_t* num_entries;          // device
  DeviceState* state;
  int64_t capacity;              // entries that fit in runs / vals
  int32_t num_tensors;
  int32_t total_blocks;          // workgroup slots of all tensors
  int32_t widest;                // of one tensor at most
  int32_t per_tensor;            // workgroups of every tensor; 0: total_blocks of them, which search
  int32_t self_scan;             // the second pass adds the block sums up itself
  unsigned long long* needs;     // device, total_blocks: one launch; null: two
  int32_t looks;                 // how often a workgroup looks for what another one leaves (see looks_for)
};

// Segments of the block-sum array handed to the scan kernel: segment s is
// [begin[s], begin[s + 1]).
struct ScanSegments {
  int32_t begin[kMaxPayloads + 1];
};

struct DecodeArgs {
  const uint16_t* runs[kMaxPayloads];
  const float* vals[kMaxPayloads];
  int64_t count[kMaxPayloads];   // entries
  ScanSegments seg;              // blocks of every payload in `sums`
  uint32_t* sums;                // positions a block covers; after the scan, the position it starts at
  float* dense;
  int64_t n;
  uint32_t* diag_flags;          // may be null
  int32_t num;                   // payloads
  int32_t block_shift;           // a block is kDecodeBlock << block_shift entries
  int32_t scanned;               // `sums` holds positions (a scan has run); 0: sizes
};

enum ScatterMode : int32_t {
  kScatterAtomicAdd = 0,
  kScatterPlainAdd = 1,
  kScatterAtomicSgd = 2,  // target += scale * value, scale = -learning rate
  kScatterPlainSgd = 3
};

// ---- launchers (dgc_compress.hip, dgc_receive.hip, dgc_wire.hip) --------------
hipError_t launch_clear_words(uint32_t* p, size_t words, hipStream_t stream);  // p[0 .. words) <- 0
int32_t norm_blocks(int64_t n);  // partial sums launch_norm leaves
hipError_t launch_norm(const float* g, int64_t n, double* partials, hipStream_t stream);
int32_t norm_shares(int64_t n);  // partial sums of launch_select with the norm
hipError_t launch_select(const SelectArgs& a, int32_t num_tensors, bool with_norm, hipStream_t stream);
hipError_t launch_band(const SelectArgs& a, const EmitBlock* blocks, int32_t num_blocks, int32_t num_tensors,
                       hipStream_t stream);
hipError_t launch_stream(const StreamArgs& a, hipStream_t stream);
hipError_t launch_ceiling(const float* a, float* b, float* c, int64_t n, int groups, hipStream_t stream);
hipError_t launch_refine(const RefineArgs& a, int32_t num_tensors, hipStream_t stream);
hipError_t launch_emit(const EmitArgs& a, int32_t num_blocks, hipStream_t stream);
int32_t compute_units();  // of the device that is current at the first call
hipError_t launch_scatter_pairs(float* dense, int64_t n, const PairPayloads& p, int32_t first,
                                int32_t num, int64_t max_count, ScatterMode mode, float scale,
                                uint32_t* diag_flags, hipStream_t stream);
// dense[idx] = 0.  `total_capacity`: pairs of a payload that the launch is sized for; `longest`: of its longest tensor
hipError_t launch_clear_regions(float* dense, int64_t n, const RegionPayloads& p, int32_t num,
                                const int64_t* out_offsets_dev, int32_t num_tensors, int64_t total_capacity,
                                int64_t longest, hipStream_t stream);

hipError_t launch_merge_regions(float* dense, const RegionPayloads& p, int32_t num, const RegionPayloads* old,
                                int32_t num_old, const int64_t* out_offsets_dev, const MergeBlock* blocks,
                                int32_t num_blocks, int64_t expected_pairs, bool scaled, float scale,
                                hipStream_t stream);
// named_only: accumulating, elements that no pair names are not stored
hipError_t launch_merge_direct(float* dense, const RegionPayloads& p, int32_t num, const RegionPayloads* old,
                               int32_t num_old, const int64_t* out_offsets_dev, const MergeBlock* parts,
                               int32_t num_parts, double expected_pairs, bool named_only, bool scaled,
                               float scale, hipStream_t stream);
hipError_t launch_merge_parts(float* dense, const RegionPayloads& p, int32_t num, const int64_t* out_offsets_dev,
                              const MergeBlock* parts, int32_t num_parts, int64_t searched_tensors, void* found, bool replace,
                              bool scaled, float scale, hipStream_t stream);
hipError_t launch_clear_parts(float* dense, const RegionPayloads& p, int32_t num, const int64_t* out_offsets_dev,
                              const MergeBlock* parts, int32_t num_parts, void* found, hipStream_t stream);
hipError_t launch_encode(EncodeArgs a, hipStream_t stream);
hipError_t launch_decode(DecodeArgs a, bool in_order, hipStream_t stream);

}  // namespace dgc

// Exported for the tests, and no part of the interface: how often this handle's workgroups look for what others leave
// before they do it themselves (0: not at all; less than zero: see looks_for).  Every number gives the same results.
extern "C" void dgc_test_set_looks(dgc_handle* h, int32_t looks);
#endif  // DGC_INTERNAL_H_
