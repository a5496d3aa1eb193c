// Launch interface of the chunk kernels (gfx950).
#pragma once
#include <hip/hip_runtime.h>
#include "common.h"

namespace mk {

// classify: digest and kind of every chunk, nothing else (first pass of a
// two-pass dump; its last pass, the gather, is k_gather in gather.hip).
enum Mode : int { kModeDump = 0, kModeDigest = 1, kModeVerify = 2, kModeRestore = 3, kModeClassify = 4 };

// One launch of the chunk engine over global chunks [g0, g1).
struct ChunkJob {
    const AllocDesc* allocs;
    uint32_t n_allocs;
    uint32_t C;                  // chunk size
    const uint32_t* amap;        // allocation of chunk g at [g], or nullptr (binary search)
    uint64_t g0, g1;
    const EngineConsts* ec;      // tables for (T, C)
    uint32_t* crc_out;           // dump / digest / classify: digest of chunk g at [g]
    uint8_t* kind_out;           // dump / classify: kind of chunk g at [g]
    const uint8_t* kind_in;      // verify / restore: kind of chunk g
    const uint32_t* ref_crc;     // verify / restore: expected digest of chunk g
    const uint32_t* prev_crc;    // dump / classify: previous digest table or nullptr
    uint8_t* slot;               // staging window (dump: written; restore: read)
    const uint64_t* off;         // restore: payload offset of chunk g
    uint64_t slot_base;          // restore: payload offset of the window start
    const uint64_t* list;        // restore: the chunks to take, ticket t the chunk list[g0 + t] (DATA chunks
                                 // only), or nullptr: chunks g0 + t
    uint64_t* status;            // dump: look-back status, indexed by g - g0
    uint64_t* wtotal;            // dump: payload bytes of the window
    unsigned long long* bad;     // verify / restore: lowest failing chunk (init ~0)
    uint32_t* err;               // internal error flag (look-back time-out)
    uint32_t epoch;              // look-back epoch of this launch (1 .. 2^22-1)
    uint32_t flags;              // kJob*
    const uint32_t* gate;        // restore / verify: when set and 0 at launch, the launch does nothing
    uint64_t* stamp;             // (of a launch's first job) device clock at the kernel's start, or nullptr
};
// verify mode: check every chunk of the range whatever its kind (the strict
// re-read after a restore), not only UNCHANGED ones
constexpr uint32_t kJobVerifyAll = 1;
// dump mode: slot is pinned host memory (plain stores in place of
// non-temporal ones, which carry 48 instead of 56 GB/s over the link)
constexpr uint32_t kJobHostSlot = 2;

// Several jobs in one persistent launch (continuous batching): the jobs'
// chunk ranges are laid end to end in one ticket space; every job keeps its
// own descriptors, tables, staging window and look-back scope, so a job's
// result does not depend on what it shares the launch with. All jobs of a
// launch use the same chunk size and tile shape (one set of LDS tables).
constexpr int kMaxJobs = 16;
struct JobList {
    ChunkJob job[kMaxJobs];
    uint64_t prefix[kMaxJobs + 1];   // ticket range of job j: [prefix[j], prefix[j+1])
    uint32_t* ticket;                // shared ticket counter, zero before launch
    uint32_t n_jobs;
    uint32_t pad;
};

// Payload offsets of every chunk of a range from the kind table.
struct OffJob {
    const AllocDesc* allocs;
    uint32_t n_allocs;
    uint32_t C;
    const uint32_t* amap;        // allocation of chunk g, or nullptr
    uint64_t n_chunks;
    const uint8_t* kind;
    uint64_t* off;               // [n_chunks]
    uint64_t* total;             // payload bytes of the range, or nullptr
    uint64_t* status;            // look-back, one word per tile
    uint32_t* ticket;
    unsigned long long* counts;  // [4]: zero, data, unchanged, invalid (zeroed before launch)
    uint32_t* err;
    uint32_t epoch;
    uint32_t pad;
    const uint32_t* rlen;        // codec layout: record length of PACKED chunk g at [g], or nullptr
    uint64_t* list;              // DATA chunks of the range in order, or nullptr
    uint64_t* n_list;            // their number (with list), or nullptr
    uint64_t* status2;           // look-back of the list positions (with list), one word per tile
    uint64_t* stamp;             // k_offsets: device clock at the kernel's start, or nullptr
    uint64_t g_base;             // the scan covers global chunks [g_base, g_base + n_chunks); off, kind
                                 // and amap are indexed globally
};

// Per-allocation combine of chunk digests into the whole-allocation CRC.
enum CombineMode : int { kCombineWrite = 0, kCombineCheck = 1, kCombineOut = 2 };
struct CombineJob {
    const AllocDesc* allocs;
    uint32_t n_allocs;
    uint32_t C;
    const uint32_t* crc;         // chunk digests (global index)
    const EngineConsts* ec;      // full_x and x2n for this C
    uint8_t* recs;               // write: AllocRec[n] (32 bytes each); check: read alloc_crc
    uint32_t* out;               // out mode: CRC of allocation a at [a]
    unsigned long long* bad;     // check mode
    int mode;
    int pad;
    uint64_t* stamp;             // device clock at the kernel's start, or nullptr
};

// What a call needs on the device before its chunk kernels, in one launch:
// the descriptors and tables brought from pinned host memory, the chunk map,
// and the words that start at a known value. Regions must not overlap; all
// are whole, aligned 32-bit words.
struct SetupJob {
    static constexpr int kMaxFills = 8, kMaxCopies = 4;
    uint64_t* stamp;             // device clock at the kernel's start, or nullptr (must not be filled here)
    const AllocDesc* src;        // pinned host descriptors
    AllocDesc* dst;              // device descriptors
    uint32_t n_allocs;
    uint32_t C;
    uint32_t* map;               // chunk map
    int n_fills, n_copies;
    struct Fill { uint32_t* p; uint64_t n; uint32_t v; uint32_t pad; } fill[kMaxFills];
    struct Copy { uint32_t* dst; const uint32_t* src; uint64_t n; } copy[kMaxCopies];
    void add_fill(void* p, uint64_t words, uint32_t v) { fill[n_fills++] = {static_cast<uint32_t*>(p), words, v, 0}; }
    void add_copy(void* d, const void* s, uint64_t bytes) {
        copy[n_copies++] = {static_cast<uint32_t*>(d), static_cast<const uint32_t*>(s), bytes / 4};
    }
};

// The end of a dump in one launch: the per-allocation combine (write mode,
// one work-group each), table words to the host image, and result words of
// earlier kernels to pinned host memory.
struct FinishJob {
    CombineJob c;
    int n_copies;
    uint32_t n_rep;              // 64-bit result words, <= 254; rep[n_rep] and [n_rep + 1] take the device
                                 // clock at the kernel's start and end
    SetupJob::Copy copy[4];
    uint64_t* rep;
    const uint64_t* rep_src;
    void add_copy(void* d, const void* s, uint64_t bytes) {
        copy[n_copies++] = {static_cast<uint32_t*>(d), static_cast<const uint32_t*>(s), bytes / 4};
    }
};

// A short full dump in one launch (k_dump_short): ticket g takes chunk g,
// ticket n_chunks + a allocation a. Everything the host prepares and
// reads is in pinned memory.
struct ShortChunk {              // 32 bytes
    const uint8_t* ptr;          // first byte of the chunk
    uint32_t len;                // valid bytes
    uint32_t full;               // len is the chunk size
    uint32_t tail_init, tail_unshift;
    uint64_t pad;
};
static_assert(sizeof(ShortChunk) == 32, "one load's worth");
struct ShortJob {
    const ShortChunk* chunks;    // pinned
    const AllocDesc* allocs;     // pinned
    uint32_t n_chunks, n_allocs;
    uint32_t C;
    uint32_t epoch;              // of status
    uint32_t* ticket;            // counter, `first` at launch (n_chunks + n_allocs more after it)
    uint32_t first, pad;
    const EngineConsts* ec;
    uint64_t* status;            // [2 n_chunks]: payload bytes of chunk g; its digest and kind
    uint8_t* payload;            // the image's, pinned like the tables:
    uint8_t* recs;
    uint32_t* crc;
    uint8_t* kind;
    uint32_t* resident;          // device copy of the digests, or nullptr
    uint64_t* rep;               // pinned, cleared by the host: payload bytes, error, device clock at the start,
                                 // with a chunk read, at the tables' start and end
};
constexpr uint32_t kShortRep = 6;
hipError_t launch_short(int T, int K, const ShortJob& job, hipStream_t s);

// A short full restore from a pinned image in one launch (k_restore_short):
// the chunks by `groups` work-groups, allocation a by work-group groups + a.
struct ShortRecord {             // 48 bytes
    uint8_t* ptr;                // first byte of the chunk
    const uint8_t* src;          // its record in the image, or nullptr: a ZERO chunk
    uint32_t len;                // valid bytes
    uint32_t full;               // len is the chunk size
    uint32_t tail_init, tail_unshift;
    uint32_t crc;                // expected digest
    uint32_t pad[3];
};
static_assert(sizeof(ShortRecord) == 48, "whole 16-byte words");
struct ShortRestoreJob {
    const ShortRecord* chunks;   // pinned
    const AllocDesc* allocs;     // pinned
    uint32_t n_chunks, n_allocs;
    uint32_t C;
    uint32_t groups;             // 1 .. n_chunks
    const EngineConsts* ec;
    const uint8_t* recs;         // the image's, pinned like its digests
    const uint32_t* crc;
    uint64_t* rep;               // pinned: device clock at the start and end of an allocation's check
    uint8_t* bad;                // pinned, [n_chunks + n_allocs], cleared by the host: 1 where a check failed
};
hipError_t launch_short_restore(int T, int K, const ShortRestoreJob& job, hipStream_t s);

// Validation of a restore inside a captured graph: *gate = 1 when the
// tables digest combined from the device's two halves equals the expected
// value, the kinds are all ZERO or DATA and the payload total equals the
// expected D; else 0 (the gated kernels then write nothing).
struct GateJob {
    const uint32_t* dig;                 // [2]: digest of AllocRec || crc[], of kind[] || pad
    uint32_t xlen;                       // x^(8 len(kind[] || pad))
    uint32_t pad;
    const unsigned long long* counts;    // [4]: zero, data, unchanged, invalid
    const uint64_t* total;               // payload total of the offsets scan
    uint64_t n_chunks;
    const uint64_t* expect;              // [2]: tables digest, D (written before each launch)
    uint32_t* gate;
};

// Digest pass over whole memory (classify and verify of chunks of at least
// kScanMinChunk bytes): group width T of the engine constants for so many
// chunks of C bytes, and the launch. job.ec must hold the constants for (T, C);
// cus: CUs the launch may fill. A wave takes 20 us for a chunk of 64 KiB by
// itself, a work-group of eight less: while there are chunks for a quarter of
// the waves at most, that counts (16 MiB: 30 us by waves, 12 by work-groups; 64
// MiB, 1024 chunks: 32 and 25; 128 MiB 38 and 42).
constexpr uint32_t kScanMinChunk = 8192;
inline int scan_width(uint32_t C, uint64_t chunks) { return C > 65536 || (C == 65536 && chunks <= 1024) ? 512 : 64; }
hipError_t launch_scan(bool verify, int T, const JobList& jl, int cus, hipStream_t s);

bool tile_supported(int T, int K);
hipError_t launch_setup(const SetupJob& job, hipStream_t s);
hipError_t launch_finish(const FinishJob& job, hipStream_t s);
// n <= 63 64-bit device words to pinned host memory; with clock, host[n]
// takes the device clock.
hipError_t launch_report(uint64_t* host, const uint64_t* dev, uint32_t n, bool clock, hipStream_t s);
hipError_t launch_gate(const GateJob& job, hipStream_t s);
hipError_t launch_chunks(int T, int K, int mode, const JobList& jl, int grid, hipStream_t s);
hipError_t chunks_occupancy(int T, int K, int mode, int* blocks_per_cu);
hipError_t launch_offsets(const OffJob& job, int grid, hipStream_t s);
hipError_t launch_combine(const CombineJob& job, hipStream_t s);
// Zero-fill of the ZERO chunks of [job.g0, job.g1) (restore; uses allocs,
// amap, ec, kind_in, ref_crc, bad and gate).
hipError_t launch_zero(const ChunkJob& job, int grid, hipStream_t s);
// launch_offsets (grid work-groups; 0: none) and launch_combine in one launch.
hipError_t launch_offsets_combine(const OffJob& off, int grid, const CombineJob& job, hipStream_t s);
hipError_t launch_chunk_map(const AllocDesc* allocs, uint32_t n_allocs, uint32_t C, uint32_t* map, hipStream_t s);
hipError_t launch_store_descs(AllocDesc* dst, const AllocDesc& a, const AllocDesc& b, hipStream_t s);
hipError_t launch_fill64(uint64_t* p, uint64_t v, uint64_t n, hipStream_t s);
hipError_t launch_fill32(uint32_t* p, uint32_t v, uint64_t n, hipStream_t s);

}  // namespace mk
