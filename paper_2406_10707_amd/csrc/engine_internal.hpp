// Internals shared by the engine's source files: the context behind the C ABI, the per-snapshot
// record, the jobs of the I/O threads, and the small helpers all of them use.
#pragma once
#include <hip/hip_runtime.h>

#include <algorithm>
#include <atomic>
#include <chrono>
#include <condition_variable>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <deque>
#include <map>
#include <memory>
#include <mutex>
#include <string>
#include <thread>
#include <vector>

#include <dirent.h>
#include <errno.h>
#include <signal.h>
#include <fcntl.h>
#include <sys/mman.h>
#include <sys/stat.h>
#include <sys/statvfs.h>
#include <unistd.h>

#include "plan.hpp"

namespace dsllm {
// t_start / t_stop (each may be null): events that receive the kernel's own start and end time
hipError_t launch_pack(const ckpt_tile *dev_tiles, uint64_t n_tiles, void *slot_base, uint64_t slot_data_off, hipStream_t stream,
                       hipEvent_t t_start = nullptr, hipEvent_t t_stop = nullptr);
hipError_t launch_scatter(const ckpt_tile *dev_tiles, uint64_t n_tiles, const void *slot_base, uint64_t slot_data_off, hipStream_t stream);
// n_blocks: how many of the n_tiles are not small (they come first)
hipError_t launch_verify_pairs(const PairTile *dev_tiles, uint64_t n_blocks, uint64_t n_tiles, uint32_t *dev_flag, hipStream_t stream);
hipError_t launch_derive_pairs(const PairTile *dev_tiles, uint64_t n_blocks, uint64_t n_tiles, hipStream_t stream);
}  // namespace dsllm

using namespace dsllm;
using Clock = std::chrono::steady_clock;


namespace dsllm {
extern thread_local std::string g_last_error;   // text behind ckpt_last_error(), per calling thread
inline int fail(int code, const std::string &msg) { g_last_error = msg; return code; }
inline double ms_between(Clock::time_point a, Clock::time_point b) { return std::chrono::duration<double, std::milli>(b - a).count(); }

// Progress lines on stderr when DSLLM_CKPT_TRACE is set in the environment (set-up stages only).
inline void trace(const char *what) {
    static const bool on = getenv("DSLLM_CKPT_TRACE") != nullptr;
    if (on) { fprintf(stderr, "[dsllm_ckpt] %s\n", what); fflush(stderr); }
}
}  // namespace dsllm

struct ckpt_plan { dsllm::Plan plan; };

namespace dsllm {

// An open checkpoint file. With retention (keep_last > 0) files, descriptors and mappings live on
// after the commit: a retired file is renamed to a hidden spare name and a later snapshot writes
// into the same pages through the same mapping, so the steady-state flush is plain memcpy.
struct FileSlot {
    std::string path;
    int fd = -1;
    uint8_t *map = nullptr;           // whole-file shared mapping when the sink is written through mmap
    uint64_t map_bytes = 0;
    uint64_t bytes = 0;               // size of the file (a spare is reused only for a snapshot of exactly this size)
    void close_all() {
        if (map) munmap(map, map_bytes);
        if (fd >= 0) ::close(fd);
        map = nullptr; fd = -1;
    }
};

struct Snap {
    uint64_t iter = 0;
    // The plan this snapshot is written with: the registration's version-1 plan, or its version-2 plan when
    // derived tensors were declared and the check on the captured state found every pair to hold. Chosen by the
    // submit thread before the first pack launch; null until then.
    const Plan *plan = nullptr;
    const ckpt_tile *dev_tiles = nullptr;   // that plan's tile table on the device
    double verify_ms = -1;                  // device time of the derivation check (-1: none)
    double window_wait_ms = 0;              // host: time the caller spent in ckpt_wait_immutable_window_end for this snapshot
    int fd = -1;
    uint8_t *map = nullptr;
    std::string tmp_path, final_path;
    std::atomic<uint64_t> chunks_left{0};
    std::atomic<bool> copies_over{false};   // one of the I/O threads has seen it
    std::atomic<int> at_tails{0};           // I/O threads that may be about to ask or wait for the tail events
    hipEvent_t ev_boundary = nullptr;
    bool submitted = false, packs_submitted = false, d2h_done = false, committed = false, window_closed = false;
    Clock::time_point t_request, t_submitted, t_committed, t_first_chunk;
    bool have_first_chunk = false;
    double call_ms = 0, backpressure_ms = 0;
    std::atomic<uint64_t> io_wait_us{0}, io_copy_us{0};   // summed over the I/O threads
    double pack_ms_sum = -1, req_to_d2h_end_ms = -1, d2h_span_ms = -1, req_to_pack_end_ms = -1;
    std::vector<uint8_t> host_capture;      // the host-resident objects as they were when the snapshot was requested
    bool straight = false;                  // the pack kernel wrote ring slot `straight_slot`: the slot's event, behind it, is this snapshot's only one
    uint64_t straight_slot = 0;
    bool head_apart = false;                // the first super-chunk was packed in two launches (its first chunk, the rest)
    int policy = CKPT_WINDOW_D2H;           // window policy in force when the snapshot was requested
    int tier2_state = CKPT_TIER2_NONE;      // ckpt_tier2_state
    double tier2_ms = -1;                   // host: copy to the second tier, open to rename
    // A failure of THIS snapshot (open, header, copy, event, chunk write, sync): its file never gets a final
    // name, whatever happens to the context-wide latch in the meantime. Guarded by the context mutex.
    bool failed = false;
    int fail_code = 0;
    std::string fail_msg;
};

struct IoJob {
    enum Kind { WRITE, READ, STOP } kind = STOP;
    std::shared_ptr<Snap> snap;   // WRITE
    int fd = -1;                  // READ
    uint64_t slot = 0, file_off = 0, nbytes = 0;
    uint64_t slot_off = 0;        // where in the slot this piece of the chunk lies
    bool ends = false;            // WRITE: after it has landed the snapshot's copies may be over (pieces of the last chunk)
    bool last = false;            // WRITE: after it has landed they are waited for (of these the last one, the first if all land together)
    hipEvent_t landed = nullptr;  // WRITE: the copy that brings this piece
    uint32_t piece = 0;           // READ: number of the piece in its chunk
};

// A chunk goes between its ring slot and the file in pieces, one job each, so that several I/O threads share it. One
// thread moves about 25 GB/s into a mapping (15 out of a file), less than half of what the link brings: with whole chunks
// a snapshot ended with one thread copying the last 64 MiB alone (2.2 ms after the last copy had landed; 0.6 in pieces),
// and a restore sent nothing to the device before 64 MiB had been read (1.1 ms; 0.4).
#ifndef DSLLM_PIECE_BYTES
#define DSLLM_PIECE_BYTES (4ull << 20)   // a multiple of 4 KiB
#endif
constexpr uint64_t kPieceBytes = DSLLM_PIECE_BYTES;
static_assert(kPieceBytes > 0 && kPieceBytes % 4096 == 0, "pieces and parts begin on the format's alignment unit (direct I/O)");
// On restore, where the copy streams take pieces in turn, pieces are a quarter of that, except for direct I/O: the link waits for the
// first one, and four threads that read 4 MiB each bring none for 0.3 ms and then four at once.
constexpr uint64_t kReadPieceBytes = kPieceBytes / 4 < 4096 ? 4096 : kPieceBytes / 4 / 4096 * 4096;
// What one copy between ring and device moves where a chunk is shared among the copy streams. One stream loses some 10 us per
// copy, two hide that from each other: 57.0 GB/s to the device in pieces of 4 MiB (one stream 50.4, whole chunks 57.6), 56.4 to the
// host in parts of 16 MiB (55.1, 57.1).
constexpr uint64_t kSendBytes = kPieceBytes, kPartBytes = 4 * kPieceBytes;
// A snapshot's only chunk goes in a copy for every 64 MiB that it has begun, all on one stream, and a copy is written while the next one lands. The
// caller's update waits for the last of them, and every copy more, with its event, takes 14 us longer: about 1 % here. (On several streams 7 us with the
// system runtime, where they land one after the other all the same, and 4 with PyTorch's, where two side by side land together.) Window (request to last copy) and request to committed file in us, as one copy / in twelve parts of 2 to 16 MiB / in these:
//    4.3 MiB  184, 194, 178   363, 241, 265       9.1 MiB  250, 289, 249   461, 331, 397       17 MiB  417, 475, 404   689, 524, 655
//     33 MiB  713, 777, 719  1231, 852, 1139       70 MiB  1425, 1506, 1441  2316, 1587, 1890   191 MiB  3683, 3777, 3721  6111, 4032, 4495
// The windows are as long beside a GEMM loop. Parts of 32 MiB: 70 MiB 1466 and 1765.
constexpr uint64_t kOneChunkStep = 16 * kPieceBytes;
inline uint64_t one_chunk_part_bytes(uint64_t chunk_bytes) {
    const uint64_t n = (chunk_bytes + kOneChunkStep - 1) / kOneChunkStep;
    return ((chunk_bytes + n - 1) / n + kAlign - 1) / kAlign * kAlign;
}
// It is written in pieces that the I/O threads share evenly: in pieces of kPieceBytes, 5.3 MiB are two, of which one thread writes the longer one
// alone (363 us to the committed file, 283 in four). At least half a MiB, for which a second thread's waking pays: 0.7 MiB, packed straight into
// the ring, 91 us in two pieces, 110 in one; 1.4 MiB 112 in three, 123 in two.
constexpr uint64_t kLeastPieceBytes = std::min<uint64_t>(512 << 10, kPieceBytes);
inline uint64_t even_piece_bytes(uint64_t part_bytes, uint64_t threads) {
    const uint64_t rounds = (part_bytes + threads * kPieceBytes - 1) / (threads * kPieceBytes), n = rounds * threads;
    return std::max(kLeastPieceBytes, ((part_bytes + n - 1) / n + kAlign - 1) / kAlign * kAlign);
}
// On restore, chunks of at least this size are sent to the device piece by piece, and each is scattered by a launch of its own as soon as it
// is there. Smaller ones are sent whole and scattered together up to this size: a launch and its wait cost the
// calling thread as much as the copy of a MiB takes. 250 MiB restored in chunks of 256 KiB 25.2 -> 17.2 ms, of 1 MiB 7.7 -> 6.4
// (with a launch for each super-chunk 17.0 and 7.3); from 8 MiB on the two are even.
#ifndef DSLLM_SCATTER_BYTES
#define DSLLM_SCATTER_BYTES (8ull << 20)
#endif
constexpr int kBoundaryEvents = 8;          // boundary events created at set-up (snapshots in flight at a time)
constexpr size_t kMaxSnapRecords = 1024;   // per-snapshot records (measurements, states) kept per context

enum SlotState : int { SLOT_FREE = 0, SLOT_BUSY = 1, SLOT_READ_DONE = 2 };

}  // namespace dsllm

struct ckpt_ctx {
    ResolvedConfig cfg;
    int device = 0;
    std::string out_dir;
    bool registered = false;
    Plan plan;

    // device resources
    uint8_t *ring = nullptr;          // pinned host
    uint64_t n_slots = 0;
    uint8_t *staging = nullptr;       // device
    uint64_t n_stage = 0;
    ckpt_tile *dev_tiles = nullptr;
    // data reduction (format version 2): declared pairs, the plan without the derived tensors, the check's tables
    DerivedPairs pairs;
    bool have_rplan = false;
    Plan rplan;
    ckpt_tile *dev_rtiles = nullptr;
    PairTile *dev_pairs = nullptr;
    uint32_t *dev_flag = nullptr, *host_flag = nullptr;   // verdict of the check: device word, pinned host word it is copied to
    hipEvent_t ev_verify_start = nullptr, ev_verify_done = nullptr, ev_derived = nullptr;
    hipStream_t pack_stream = nullptr;
    std::vector<hipStream_t> dma;
    std::vector<hipEvent_t> ev_slot;                      // per ring slot: copy into or out of the slot done
    std::vector<std::vector<hipEvent_t>> ev_sent;         // restore in chunks that may be sent on several streams, [dma stream - 1][slot]: the other streams' copies
    std::vector<std::vector<hipEvent_t>> ev_part;         // [chunks from the end][part]: part of one of a snapshot's last chunks
    // restore: what the stream had to copy when the slot's chunk was sent (whichever stream that is, if it is always one)
    hipEvent_t sent_event(size_t stream, uint64_t slot) const { return stream == 0 || ev_sent.empty() ? ev_slot[slot] : ev_sent[stream - 1][slot]; }
    bool shares_last_chunks() const { return dma.size() > 1 && cfg.dma_chunk_bytes > dsllm::kPartBytes; }
    std::vector<hipEvent_t> ev_pack_start, ev_pack_end, ev_packed;   // per super-chunk: the kernel's start and end (timing), its completion in the pack stream (ordering)
    std::vector<std::vector<hipEvent_t>> ev_stage_done;   // [stage slot][dma stream]
    std::vector<hipEvent_t> ev_job_tail;                  // per dma stream
    // The events that the snapshot's copies end with. A slot's event is not recorded again before the slot has been written; ev_job_tail are
    // the next snapshot's as soon as the copies are over.
    size_t tails(const Snap *s) const { return s->straight ? 1 : dma.size(); }
    hipEvent_t tail(const Snap *s, size_t k) const { return s->straight ? ev_slot[s->straight_slot] : ev_job_tail[k]; }
    hipEvent_t ev_first_copy = nullptr, ev_user = nullptr;
    hipEvent_t ev_packed_head = nullptr;                  // the first chunk of a snapshot is in staging
    hipEvent_t ev_head_end = nullptr, ev_rest_start = nullptr;   // timing of the first super-chunk's two launches, between ev_pack_start[0] and ev_pack_end[0]
    hipEvent_t ev_scattered = nullptr;                    // restore: what the pack stream held before it has read staging
    uint8_t *hdr_buf = nullptr;                           // 4 KiB-aligned scratch for header writes
    uint64_t ring_next = 0;                               // global chunk counter -> ring slot
    double init_d2h_gbps = -1;                            // one ring slot copied device-to-host at set-up, timed (-1: could not be measured)

    // threads and queues
    std::mutex mu;
    std::condition_variable cv_submit, cv_io, cv_state;   // submit queue / io queue / any state change
    std::deque<std::shared_ptr<Snap>> submit_q;
    std::deque<IoJob> io_q;
    std::vector<int> slot_state;
    std::vector<uint32_t> slot_pieces_left;               // pieces of the slot's chunk still to be written or read
    std::vector<std::vector<uint8_t>> slot_piece_read;    // restore: which pieces of the slot's chunk have been read
    bool stopping = false;
    std::thread submit_thread;
    std::vector<std::thread> io_threads;
    std::map<uint64_t, std::shared_ptr<Snap>> snaps;
    std::shared_ptr<Snap> last_snap;       // most recent request
    std::shared_ptr<Snap> prev_job;        // submit thread: job before the current one
    int async_code = 0;
    std::string async_err;
    bool restoring = false;
    // retention: committed iterations in commit order, and retired files whose pages are reused
    std::deque<uint64_t> committed_iters;
    std::vector<FileSlot> spares;
    std::map<uint64_t, FileSlot> kept;     // committed files that still carry their names
    uint64_t spare_seq = 0;
    // second tier: committed files are copied on to a slower, durable directory by a thread of their own
    bool tier2_on = false, tier2_enabling = false, tier2_direct = false, tier2_stop = false;
    std::string tier2_dir;
    int tier2_threads = 4, tier2_keep = 1, tier2_mode = CKPT_TIER2_NEWEST;
    std::thread tier2_thread, tier2_unlinker;   // the latter is touched by the second-tier thread only (and by destroy after joining it)
    std::condition_variable cv_tier2;
    std::shared_ptr<Snap> tier2_waiting;   // newest committed snapshot not yet picked up (latest wins)
    std::shared_ptr<Snap> tier2_active;    // being copied: its first-tier file must not be recycled
    bool tier2_removals_pending = false;   // superseded second-tier files are still being unlinked
    bool tier2_retire_after = false;       // the active file fell out of the newest keep_last meanwhile
    std::deque<uint64_t> tier2_files;      // iterations present in the second tier, oldest first
    int tier2_code = 0;                    // first failure of a second-tier copy, reported by ckpt_wait_second_tier
    std::string tier2_err;

    std::vector<hipEvent_t> ev_boundary_free;             // boundary events, created at set-up, handed out per request

    void latch(int code, const std::string &msg) {
        std::lock_guard<std::mutex> lk(mu);
        if (async_code == 0) { async_code = code; async_err = msg; }
        cv_state.notify_all();
    }
    // Marks one snapshot as failed (first failure wins) and latches the error for the caller's next call.
    void fail_snapshot(dsllm::Snap *s, int code, const std::string &msg) {
        std::lock_guard<std::mutex> lk(mu);
        if (!s->failed) { s->failed = true; s->fail_code = code; s->fail_msg = msg; }
        if (async_code == 0) { async_code = code; async_err = msg; }
        cv_state.notify_all();
    }
};

#define HIP_TRY(ctx, expr)                                                                     \
    do {                                                                                       \
        hipError_t e_ = (expr);                                                                \
        if (e_ != hipSuccess) return fail(CKPT_EHIP, std::string(#expr) + ": " + hipGetErrorString(e_)); \
    } while (0)

namespace dsllm {
// size of the file a snapshot of this registration is expected to have (what spare files are made for)
inline uint64_t expected_file_bytes(const ckpt_ctx *c) { return c->have_rplan ? c->rplan.file_bytes() : c->plan.file_bytes(); }
inline std::string file_name_for(const std::string &dir, uint64_t iter) {
    char buf[64];
    snprintf(buf, sizeof buf, "/ckpt_iter%020llu.dsl", (unsigned long long)iter);
    return dir + buf;
}

// Makes a rename in `dir` durable: the directory entry itself has to reach the disk.
inline bool fsync_dir(const std::string &dir, std::string *err) {
    int fd = open(dir.c_str(), O_RDONLY | O_DIRECTORY);
    if (fd < 0) { *err = dir + ": open: " + strerror(errno); return false; }
    const bool ok = fsync(fd) == 0;
    if (!ok) *err = dir + ": fsync: " + strerror(errno);
    close(fd);
    return ok;
}

inline bool pwrite_all(int fd, const uint8_t *p, uint64_t n, uint64_t off, std::string *err) {
    while (n) {
        size_t want = n > (1ull << 30) ? size_t(1ull << 30) : size_t(n);
        ssize_t w = pwrite(fd, p, want, off_t(off));
        if (w < 0) { if (errno == EINTR) continue; *err = std::string("pwrite: ") + strerror(errno); return false; }
        p += w; off += uint64_t(w); n -= uint64_t(w);
    }
    return true;
}

inline bool pread_all(int fd, uint8_t *p, uint64_t n, uint64_t off, std::string *err) {
    while (n) {
        size_t want = n > (1ull << 30) ? size_t(1ull << 30) : size_t(n);
        ssize_t r = pread(fd, p, want, off_t(off));
        if (r < 0) { if (errno == EINTR) continue; *err = std::string("pread: ") + strerror(errno); return false; }
        if (r == 0) { *err = "pread: unexpected end of file"; return false; }
        p += r; off += uint64_t(r); n -= uint64_t(r);
    }
    return true;
}


// io_threads.cpp
void io_thread_main(ckpt_ctx *c);
void read_piece(ckpt_ctx *c, const IoJob &job, uint8_t *bounce);
void retire_locked(ckpt_ctx *c, uint64_t iter);
// second_tier.cpp
void tier2_offer_locked(ckpt_ctx *c, const std::shared_ptr<Snap> &sp);
void tier2_thread_main(ckpt_ctx *c);
// submit.cpp
void submit_thread_main(ckpt_ctx *c);
// pack_image.hip
int pack_image_setup(hipStream_t stream);
// engine.cpp
int take_async_error(ckpt_ctx *c);
bool preallocate_file(const std::string &path, uint64_t bytes, int n_threads, bool map_it, bool o_direct, FileSlot *out, std::string *err);
}  // namespace dsllm

