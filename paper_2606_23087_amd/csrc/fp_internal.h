// Internal layout shared by the host pool code and the HIP kernels of
// libflowpool. Not part of the public ABI (see include/flowpool.h).
#pragma once

#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

namespace fp {

// Device sample descriptor, one per resident sample slot (48 bytes).
// The variable-length parts live in the metadata arena at byte offsets:
//   page_off: uint64 GVA per page, in visual-row order      [n_pages]
//   img_off : int32 pairs (placeholder position, rows)       [n_img]
//   text_off: int32 text token ids                            [n_text]
struct alignas(16) SampleDesc {
  int32_t len;      // n_text + n_vis
  int32_t n_text;
  int32_t n_img;
  int32_t n_vis;
  int64_t page_off;
  int64_t img_off;
  int64_t text_off;
  int32_t n_pages;
  int32_t pad;
};
static_assert(sizeof(SampleDesc) == 48, "descriptor layout");

// Page-table entry: device-visible address of the physical page, low bits
// used as flags (page addresses are at least 16-byte aligned).
constexpr uint64_t PTE_VALID = 1ull;
constexpr uint64_t PTE_HOST = 2ull;
constexpr uint64_t PTE_ADDR_MASK = ~0xFull;

constexpr int kBlock = 256;          // threads per workgroup for all kernels
constexpr int kPackBlock = 256;      // threads per k_pack workgroup
constexpr int kVecsPerThread = 3;    // 16-byte vectors each k_pack thread moves (12 KiB chunks)
constexpr int kChunkVecs = kPackBlock * kVecsPerThread;   // output vectors per k_pack workgroup
// Rows of at least this many bytes are packed in 8 KiB chunks (2 vectors per
// thread) instead: measured faster from H 5120 up, slower at H 3584 and 4096.
constexpr int kSmallChunkRowBytes = 10240;
// The last chunks of a pack are smaller, so the final workgroups finish
// sooner and the launch drains faster: one wave of resident workgroups (CUs x
// kPackPerCU) gets chunks of kTail1Vecs (the full size when rows take 8 KiB
// chunks), half a wave then kTail2Vecs.
constexpr int kPackPerCU = 8;        // k_pack workgroups resident per CU (occupancy 8)
constexpr int kTail1Vecs = 512;
constexpr int kTail2Vecs = 256;
constexpr int kBuckets = 64;         // row buckets of the run index at most
constexpr int kMinBuckets = 16;      // and at least, in a table passed by value that could not hold kBuckets
// A pack of more samples or runs than these is not captured into a graph
// (each such run table fits the kernel arguments with kBuckets buckets).
constexpr int kCaptureSamples = 32;
constexpr int kCaptureRuns = 160;
constexpr int kWaveRows = 16;        // rows per wave resolved with scalar loads in k_pack
constexpr int kMaxPackSamples = 1024;  // per microbatch (bounds the staged run table)
constexpr int kMaxPackImages = 1024;

// A run is a maximal stretch of packed rows of one sample that come from one
// place: text rows (ids read from the sample's text list) or image rows (the
// images between two text rows, which are consecutive in the sample's page
// list). The host lists a microbatch's runs in row order, so resolving a row
// is finding its run and one or two indexed loads. Metadata-arena offsets are
// kept as word indexes, so the arena is limited to kMaxMetaBytes.
struct alignas(16) PackRun {
  int32_t end;        // one past the run's last row
  int32_t head;       // first row of the run's sample; bit 31 set for a text run
  int32_t vdelta;     // image run: visual index of row r is r + vdelta
  int32_t word;       // text run: the id of row r is 32-bit word word + r of the
                      // arena; image run: the sample's page GVAs start at
                      // 64-bit word `word`, or, when its pages have
                      // consecutive GVAs, -1 - (page number of its first page)
};
static_assert(sizeof(PackRun) == 16, "PackRun layout");
constexpr int32_t kTextRun = INT32_MIN;
// A bit of PackArgs::tier_mask beside the two tier bits: chunks holding
// embedding-table rows read with plain loads, which let the device's 256 MB
// memory-side cache keep table rows between reads. Set for tables of at most
// kPlainTableMaxBytes: over uniform random rows, plain loads gather 9 % faster
// than non-temporal ones from a 1.09 GB table, break even near 3 GB, and
// are 1.5 % slower from a 4.3 GB one.
constexpr int32_t kTablePlainLoads = 4;
constexpr int64_t kPlainTableMaxBytes = 5ll << 29;   // 2.5 GiB
constexpr int64_t kMaxMetaBytes = 1ll << 33;

// The run table: the samples' lengths, their runs, and the bucket index: for
// each row bucket b a copy of the run holding row b << shift, then that run's
// index (16 bits), so a row of the same run is resolved with one load, and a
// later row steps on from there. Byte offsets of the parts; size 0: no table.
struct RunTable {
  int32_t runs, bucket_runs, bucket_index, size;
  int32_t n_buckets, shift;   // buckets hold 2^shift rows
};

// What the pack kernel reads, passed by value. The run table follows the
// scalar fields; kernel arguments are captured at launch, so a microbatch
// whose table fits needs no copy of it. A larger one is copied to device
// memory first. The table's room is a template parameter: PackArgs is the
// general form, PackArgsSmall a compact one for microbatches of a few
// samples: a launch with 0.8 KB of arguments takes 3.1 us of host time and 12
// until its completion is seen on an idle stream, one with 4 KB 3.9 and 20.
template <int kBytes>
struct PackArgsT {
  const uint8_t* meta;        // device metadata arena
  const uint64_t* pte;        // device page table, index = (gva - gva_start) / page_bytes
  uint64_t gva_start;
  const uint8_t* table;       // embedding table (may be null when no text row is copied)
  uint8_t* out;               // packed rows
  int32_t* cu;                // cu_seqlens or null
  int32_t* pos;               // position ids or null
  int32_t off_runs;           // byte offsets from the table's start: the runs,
  int32_t off_brun;           // the bucket runs and the bucket index
  int32_t off_bucket;
  int32_t bucket_shift;       // buckets hold 2^bucket_shift rows
  int32_t n;                  // samples
  int32_t n_tokens;           // total rows
  int32_t row_bytes;
  int32_t page_tokens;
  int32_t tier_mask;          // FP_TIER_MASK_* bits, plus kTablePlainLoads
  uint64_t pt_mul;            // v / page_tokens == (v * pt_mul) >> pt_shift for v < 2^31
  uint64_t pb_mul;            // d / page_bytes == umulhi64(d, pb_mul) >> pb_shift for d < 2^52
  int32_t pt_shift;
  int32_t pb_shift;
  alignas(16) uint8_t run_table[kBytes];
  static constexpr int kTableBytes = kBytes;
};
using PackArgs = PackArgsT<3840>;
using PackArgsSmall = PackArgsT<704>;
// The pack's kernel arguments, 64 bytes of leading scalars (preloaded into
// registers) and this struct, stay within 4 KiB.
static_assert(sizeof(PackArgs) + 64 <= 4096, "kernel arguments stay within 4 KiB");
static_assert(offsetof(PackArgs, run_table) == offsetof(PackArgsSmall, run_table), "same scalar fields");

// A pack launch: the kernel's arguments and, host side, its geometry.
struct PackPlan {
  PackArgs a;
  const uint8_t* staged;      // staged run table, or null = the one in `a`
  bool small;                 // launch with PackArgsSmall (its table copied from `a`)
  int32_t max_chunk_rows;     // rows one chunk can touch
  int32_t g0, g1;             // workgroups [0, g0): full chunks; [g0, g1): kTail1Vecs; then kTail2Vecs
  int32_t t1, t2;             // first vectors of the two tail stages (t1 = g0 * full chunk)
  int32_t vpt;                // vectors per thread of a full chunk (2 or kVecsPerThread)
  uint64_t div_mul;           // e / (row_bytes/16) == (e * div_mul) >> div_shift for e < 2^31
  int32_t div_shift;
};

// Division constants of a pool (host-computed once): for e < 2^31,
// e / (row_bytes / 16) == (e * div_mul) >> div_shift and
// e / page_tokens == (e * pt_mul) >> pt_shift; for d < 2^52,
// d / page_bytes == umulhi64(d, pb_mul) >> pb_shift.
struct Divisors {
  uint64_t div_mul, pt_mul, pb_mul;
  int32_t div_shift, pt_shift, pb_shift;
};

// The producer's write of one sample: its visual rows (contiguous at `vis`)
// are copied into its pages, cut into chunks like a pack, and its metadata
// (page list, image list, text ids) and descriptor go from pinned host memory
// and the kernel arguments into the arena, in one launch. The numbers of up to
// kInlinePages scattered pages travel in the arguments (WriteArgs); of
// consecutive pages the first alone does, and a longer scattered list is read
// from the staging buffer (both WriteArgsSmall).
template <int kCapacity>
struct WriteArgsT {
  SampleDesc desc;            // descriptor to publish into the table
  SampleDesc* desc_table;
  const uint8_t* stage;       // the metadata block in pinned host memory (16-byte aligned)
  uint8_t* meta;              // where it goes in the device arena
  const uint64_t* pte;
  int32_t slot;
  int32_t meta_vecs;          // 16-byte vectors of the metadata block
  int32_t row_bytes;
  int32_t page_tokens;
  int32_t staged_pages;       // WriteArgsSmall: page GVAs are the block's first words, else consecutive
  uint64_t gva_start;
  uint64_t pt_mul, pb_mul;    // division constants (as in PackArgs)
  int32_t pt_shift, pb_shift;
  uint32_t page[kCapacity];   // page numbers (WriteArgsSmall: of page 0)
  static constexpr int kPages = kCapacity;
};
// A list costs host time to fill and to pass: the C call of a write takes 3.93
// us with 4 scattered pages and 3.87 with 4 consecutive ones, 5.01 and 4.69
// with 180. So writes whose page numbers need no list take the small form; a
// list longer than this is read from the staging buffer (4.86 and 4.73 us with
// 250 pages), by a kernel long enough to hide the reads across the link.
constexpr int kInlinePages = 192;
using WriteArgs = WriteArgsT<kInlinePages>;
using WriteArgsSmall = WriteArgsT<1>;
static_assert(offsetof(WriteArgs, page) == offsetof(WriteArgsSmall, page), "same scalar fields");
// Metadata vectors one workgroup of a write uploads.
constexpr int kMetaVecs = kPackBlock * 4;

struct WritePlan {
  WriteArgs a;
  const uint8_t* vis;         // producer rows, or null
  bool inline_pages;          // launch with WriteArgs, else WriteArgsSmall
  int32_t max_chunk_rows;     // rows one chunk can touch
  uint64_t div_mul;           // e / (row_bytes/16) == (e * div_mul) >> div_shift
  int32_t div_shift;
};

// A migration's work list, in pinned host memory: per sample its new page
// list, then the pieces to copy.
struct alignas(16) MigrateList {
  int64_t words_at;           // byte offset of the list in the work list's buffer
  int64_t meta_off;           // where it goes in the arena; also the descriptor's new page_off
  int32_t n_words;
  int32_t slot;
  int64_t pad;
};
struct alignas(16) MigratePiece {
  uint64_t src, dst;          // device-visible addresses
  uint32_t vecs;              // 16-byte vectors to copy, at most kMigratePieceVecs
  uint32_t pad;
  uint64_t pad1;
};
// Threads of a workgroup (one wave), workgroups that copy pieces, by the target
// tier, and vectors of a piece one moves per step (see k_migrate).
constexpr int kMigrateBlock = 64;
constexpr int kMigrateGrid[2] = {21, 40};
constexpr uint32_t kMigrateVecs = 64 * 4;
constexpr int64_t kMigratePieceVecs = 1 << 30;
// A page of at least this many steps is a piece of its own, of which at most
// the last step moves less than a whole one. Smaller pages that are adjacent in
// both tiers are taken together and cut into pieces of one step.
constexpr int kMigratePageSteps = 8;

// A run of adjacent pages of at least this many bytes is one copy by the DMA
// engines instead, which leave the CUs to the packs beside them but take some 10
// us a copy. 134 MB to HBM / to the host tier, by copies and by the kernel: in
// runs of 8 MiB 2.52 / 2.53 and 2.42 / 2.39 ms alone, 2.75 / 2.55 and 3.44 / 3.52
// beside a stream of packs (38.7 / 38.5 us each and 39.0 / 38.6); in runs of 32 MiB
// 2.40 / 2.41 and 2.40 / 2.38 alone, 2.41 / 2.42 and 3.44 / 3.55 beside packs. In
// runs of 4 MiB copies would take 17 % longer alone and gain 4 % beside packs.
constexpr int64_t kMigrateCopyBytes = 8 << 20;

struct MigrateArgs {
  const uint8_t* stage;       // n_lists MigrateList, the lists' words, n_pieces MigratePiece
  uint8_t* meta;
  SampleDesc* desc_table;
  int64_t pieces_at;          // byte offset of the pieces
  uint32_t n_pieces;
  uint32_t steps_per_piece;   // kMigrateVecs each, of the longest piece
  int32_t n_lists;
  int32_t tier;               // target
};

// The slots of a plan's samples travel in the cost kernel's arguments up to
// this many (within 4 KiB with the other arguments), so that the kernel does
// not read them across the link.
constexpr int kCostSlots = 960;
struct CostArgs {
  const SampleDesc* desc;
  const int32_t* slots;       // pinned host memory, or null = `slot`
  int64_t* out;
  int64_t k;
  int32_t n;
  int32_t slot[kCostSlots];
};
static_assert(sizeof(CostArgs) <= 4096, "kernel arguments stay within 4 KiB");

size_t pack_lds_bytes(const PackPlan& pl);
Divisors make_divisors(int64_t row_bytes, int64_t page_tokens, uint64_t page_bytes);
// Chunk geometry of a pack (g0, g1, t1, t2) for a device with n_cu compute units.
void pack_chunks(PackPlan* pl, int n_cu);
// Launches a pack; `done`, if not null, completes with its kernel.
hipError_t launch_pack(const PackPlan& pl, hipStream_t stream, hipEvent_t done);
// Launches a write; `done` completes with its kernel.
hipError_t launch_write(const WritePlan& pl, int n_cu, hipStream_t stream, hipEvent_t done);
// Launches a migration; `done` completes with its kernel.
hipError_t launch_migrate(const MigrateArgs& a, hipStream_t stream, hipEvent_t done);
// Measurement aids with the pack's geometry: a plain copy of `vecs` 16-byte
// vectors (chunks sized as for rows of row_bytes), and a gather of n_rows
// rows of row_bytes from the device addresses rows_src[] into consecutive
// rows of dst.
hipError_t launch_copy(const void* src, void* dst, int64_t vecs, int64_t row_bytes, int n_cu, hipStream_t stream);
hipError_t launch_gather(const uint64_t* rows_src, int32_t n_rows, int64_t row_bytes, void* dst, int n_cu,
                         hipStream_t stream);
// Costs of the samples in slots[0, n) (host memory) into out_cost (device-visible). More than
// kCostSlots of them are read through slots_dev, the GPU's view of the same array in pinned memory.
// `done` completes with the kernel.
hipError_t launch_cost(const SampleDesc* desc, const int32_t* slots, const int32_t* slots_dev, int32_t n, int64_t k,
                       int64_t* out_cost, hipStream_t stream, hipEvent_t done);

}  // namespace fp
