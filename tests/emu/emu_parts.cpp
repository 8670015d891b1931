// Snapshots in parts and restores of files larger than the ring, on the CPU model of streams and events (hip/hip_runtime.h).
//   end      a slow sink: once its copies have landed, a snapshot says so, and the next one starts, while its last chunk is
//            still being written
//   restore  a restore hands a chunk's copies to the device while those of the chunk before it are under way, also when the
//            ring's slots come round again
//   events   a context has the events that its chunks and streams need
//   one      a shard of one chunk, or two, whose copies come late, one after the other: no piece is written before all of it has landed; a
//            single chunk has a copy for every sixteen pieces' bytes, each of two chunks one for every four
//   straight a shard that is packed straight into its slot and written in pieces, behind a slow sink: the file is committed
//            while the next snapshot, which the end of these copies has let start, is held on its stream
//   late     the thread with the last piece is held right before it asks for the end of the copies, and another one says that they are over:
//            it does not wait for the next snapshot's
//   emu_parts <dir> end|restore|events|one|straight|late [<chunk bytes> <ring slots>]
#include <algorithm>
#include <atomic>
#include <chrono>
#include <cstdio>
#include <cstdlib>
#include <functional>
#include <map>
#include <mutex>
#include <string>
#include <thread>
#include <vector>

#include <sys/uio.h>
#include <unistd.h>

#include "../../include/ckpt.h"
#include "hip/hip_runtime.h"

thread_local dim3 threadIdx, blockIdx, blockDim, gridDim;
static std::function<void(off_t)> g_before_write;
ssize_t emu_pwrite(int fd, const void *buf, size_t n, off_t off) {
    if (g_before_write) g_before_write(off);
    struct iovec iov = {const_cast<void *>(buf), n};
    return pwritev(fd, &iov, 1, off);
}
#ifndef DSLLM_PIECE_BYTES
#define DSLLM_PIECE_BYTES (4ull << 20)
#endif
#define REQUIRE(x) do { if (!(x)) { printf("FAILED line %d: %s (%s)\n", __LINE__, #x, ckpt_last_error()); exit(1); } } while (0)

// waits until it holds, five seconds at most: no wait here can hang the test
template <class F> static bool comes_true(F f) {
    for (int i = 0; i < 5000; i++) {
        if (f()) return true;
        std::this_thread::sleep_for(std::chrono::milliseconds(1));
    }
    return false;
}

struct Run {
    std::vector<std::vector<uint8_t>> t;
    std::vector<std::string> names;
    std::vector<int64_t> shapes;
    ckpt_ctx *ctx = nullptr;
    ckpt_layout lay;
    hipStream_t compute;

    Run(const std::string &dir, const std::vector<uint64_t> &sizes, uint64_t chunk, uint64_t slots, int io_threads, int policy = CKPT_WINDOW_D2H) {
        for (uint64_t n : sizes) { t.emplace_back((n + 15) / 16 * 16); shapes.push_back(int64_t(n)); names.push_back("t" + std::to_string(names.size())); }
        std::vector<ckpt_tensor_desc> descs;
        for (size_t k = 0; k < t.size(); k++) {
            ckpt_tensor_desc d{};
            d.name = names[k].c_str(); d.dtype = CKPT_U8; d.ndim = 1; d.shape = &shapes[k]; d.dev_ptr = t[k].data(); d.nbytes = uint64_t(shapes[k]);
            descs.push_back(d);
        }
        ckpt_config cfg{};
        cfg.out_dir = dir.c_str();
        cfg.host_ring_bytes = slots * chunk;
        cfg.dma_chunk_bytes = chunk;
        cfg.pack_superchunk_bytes = 2 * chunk;
        cfg.n_dma_streams = 2;
        cfg.n_io_threads = io_threads;
        cfg.io_mode = CKPT_IO_PWRITE;
        cfg.window_policy = policy;
        REQUIRE(ckpt_init(&cfg, &ctx) == CKPT_OK);
        REQUIRE(ckpt_register_tensors(ctx, descs.data(), descs.size()) == CKPT_OK);
        REQUIRE(ckpt_get_layout(ctx, &lay) == CKPT_OK);
        hipStreamCreateWithFlags(&compute, hipStreamNonBlocking);
    }
    static uint8_t byte(uint64_t k, uint64_t j, uint64_t it) { return uint8_t((j * 2654435761ull + k * 40503ull + it * 97ull) >> 8); }
    void snapshot(uint64_t it) {
        emu_submit(compute, [this, it] { for (size_t k = 0; k < t.size(); k++) for (uint64_t j = 0; j < uint64_t(shapes[k]); j++) t[k][j] = byte(k, j, it); });
        REQUIRE(ckpt_snapshot_async(ctx, it, compute) == CKPT_OK);
    }
    std::string file(uint64_t it) {
        char name[4096];
        REQUIRE(ckpt_file_name(ctx, it, name, sizeof name) == CKPT_OK);
        return name;
    }
    void restored(uint64_t it) {
        emu_submit(compute, [this] { for (auto &x : t) std::fill(x.begin(), x.end(), 0xA5); });
        uint64_t got = 0;
        REQUIRE(ckpt_restore(ctx, file(it).c_str(), compute, &got) == CKPT_OK && got == it);
        hipStreamSynchronize(compute);
        for (size_t k = 0; k < t.size(); k++) for (uint64_t j = 0; j < uint64_t(shapes[k]); j++) REQUIRE(t[k][j] == byte(k, j, it));
    }
    ~Run() {
        REQUIRE(ckpt_destroy(ctx) == CKPT_OK);
        hipStreamDestroy(compute);
    }
};

// One I/O thread. It is held at the first piece of the last chunk until the copies are over, and at the second one until the
// next snapshot, which waits for the end of these copies, has been submitted.
static void end_of_copies(const std::string &dir) {
    const uint64_t chunk = 128 << 10;
    Run r(dir, {200000, 100000, 40000}, chunk, 8, 1);
    const off_t last = off_t(r.lay.header_bytes + (r.lay.n_chunks - 1) * chunk);
    REQUIRE(r.lay.n_chunks == 3 && r.lay.data_bytes > 2 * chunk + 20000);
    std::atomic<bool> landed{false}, first{false}, done{false};
    ckpt_stats st;
    g_before_write = [&](off_t off) {
        if (off < last || done) return;
        if (!first.exchange(true)) { REQUIRE(comes_true([&] { return landed.load(); })); return; }
        done = true;
        REQUIRE(ckpt_get_stats(r.ctx, 1, &st) == CKPT_OK && st.d2h_done == 1 && st.committed == 0);
        REQUIRE(comes_true([&] { return ckpt_get_stats(r.ctx, 2, &st) == CKPT_OK && st.host_submit_ms >= 0; }));
    };
    r.snapshot(1);
    REQUIRE(ckpt_wait_immutable_window_end(r.ctx, r.compute, 1) == CKPT_OK);     // returns when the last copy has landed
    r.snapshot(2);
    landed = true;
    REQUIRE(ckpt_flush(r.ctx, CKPT_ITER_ALL) == CKPT_OK);
    REQUIRE(done);
    g_before_write = nullptr;
    r.restored(1);
    r.restored(2);
}

// A copy is held until one of the next chunk has been handed over. In between the ends, chunks of more than sixteen pieces go as a
// whole then: one copy each.
static std::mutex g_copies;
static uint64_t g_chunk = 0, g_handed = 0;
static std::map<const void *, uint64_t> g_chunk_of;
static std::vector<int> g_copies_of;
static std::atomic<bool> g_alone{false};

static void on_copy(const void *src, size_t n, hipMemcpyKind kind, bool starts) {
    if (kind != hipMemcpyHostToDevice) return;
    std::unique_lock<std::mutex> lk(g_copies);
    if (!starts) {
        g_chunk_of[src] = g_handed / g_chunk;
        g_copies_of[g_handed / g_chunk]++;
        g_handed += n;
        return;
    }
    const uint64_t ch = g_chunk_of[src];
    lk.unlock();
    if (ch + 1 < g_copies_of.size() && !g_alone && !comes_true([&] { std::lock_guard<std::mutex> l(g_copies); return g_handed > (ch + 1) * g_chunk; })) g_alone = true;
}

static void restore(const std::string &dir, uint64_t chunk, uint64_t slots) {
    Run r(dir, {3 * chunk + 777, 100, 5 * chunk, 2 * chunk + 4097}, chunk, slots, 3);
    r.snapshot(1);
    REQUIRE(ckpt_wait_immutable_window_end(r.ctx, r.compute, 0) == CKPT_OK);
    REQUIRE(ckpt_flush(r.ctx, 1) == CKPT_OK);
    for (int rep = 0; rep < 2; rep++) {
        g_chunk = chunk;
        g_handed = 0;
        g_copies_of.assign(r.lay.n_chunks, 0);
        g_emu_copy_hook = on_copy;
        r.restored(1);
        g_emu_copy_hook = nullptr;
        REQUIRE(!g_alone && g_handed == r.lay.data_bytes);
        for (uint64_t ch = 0; ch < r.lay.n_chunks; ch++)
            REQUIRE(g_copies_of[ch] >= 1 && (chunk <= 16 * DSLLM_PIECE_BYTES || ch < 2 || ch + 1 == r.lay.n_chunks || g_copies_of[ch] == 1));
    }
}

static int events_of(const std::string &dir, uint64_t chunk, uint64_t slots, int streams) {
    ckpt_config cfg{};
    cfg.out_dir = dir.c_str();
    cfg.host_ring_bytes = slots * chunk;
    cfg.dma_chunk_bytes = chunk;
    cfg.pack_superchunk_bytes = 2 * chunk;
    cfg.n_dma_streams = streams;
    ckpt_ctx *ctx = nullptr;
    const int before = g_emu_events_created;
    REQUIRE(ckpt_init(&cfg, &ctx) == CKPT_OK);
    const int made = g_emu_events_created - before;
    REQUIRE(ckpt_destroy(ctx) == CKPT_OK);
    return made;
}

// with the library's own piece sizes
static void events(const std::string &dir) {
    for (int streams : {1, 2, 3}) {
        REQUIRE(events_of(dir, 256 << 10, 96, streams) - events_of(dir, 256 << 10, 32, streams) == 64);          // one for every slot
        REQUIRE(events_of(dir, 8 << 20, 6, streams) - events_of(dir, 8 << 20, 2, streams) == 4 * streams);       // sent on several streams
    }
    REQUIRE(events_of(dir, 40 << 20, 2, 1) == events_of(dir, 256 << 10, 2, 1));                                  // parts of the last chunks:
    REQUIRE(events_of(dir, 40 << 20, 2, 2) - events_of(dir, 16 << 20, 2, 2) == 3 * 3);                           // three chunks, three parts
}

// Policy PACK: a chunk this small would be packed straight into its slot under the other one. Sizes that leave parts of every
// length in pages, and pieces that don't divide them.
static std::atomic<int> g_copies_made{0};
static void one_chunk(const std::string &dir, uint64_t chunk) {
    for (uint64_t pages : {chunk / 4096, chunk / 4096 - 1, chunk / 4096 * 3 / 4, chunk / 8192 + 3, chunk / 16384 + 1, chunk / 4096 + 3, chunk / 2048 - 1}) {
        Run r(dir, {4096 * pages - 4096 * 2 - 5, 4096, 77}, chunk, 2, 3, CKPT_WINDOW_PACK);
        const uint64_t data = 4096 * pages, part = (data > chunk ? 4 : 16) * DSLLM_PIECE_BYTES;
        REQUIRE(r.lay.data_bytes == data && r.lay.n_chunks == (data + chunk - 1) / chunk);
        uint64_t copies = 0;
        for (uint64_t at = 0; at < data; at += chunk) copies += chunk > 4 * DSLLM_PIECE_BYTES ? (std::min(chunk, data - at) + part - 1) / part : 1;
        for (uint64_t it = 1; it <= 2; it++) {
            g_copies_made = 0;
            g_emu_copy_hook = [](const void *, size_t, hipMemcpyKind kind, bool starts) {
                if (kind == hipMemcpyDeviceToHost && starts) { g_copies_made++; std::this_thread::sleep_for(std::chrono::milliseconds(5)); }
            };
            r.snapshot(it);
            REQUIRE(ckpt_wait_immutable_window_end(r.ctx, r.compute, 0) == CKPT_OK);
            REQUIRE(ckpt_flush(r.ctx, it) == CKPT_OK);
            g_emu_copy_hook = nullptr;
            REQUIRE(uint64_t(g_copies_made) == copies);
        }
        r.restored(1);
        r.restored(2);
    }
}

// One I/O thread, held at its first piece until the next snapshot has been submitted; the next snapshot's stream is held
// until the first file has been committed.
static std::atomic<hipStream_t> g_compute{nullptr};
static std::atomic<bool> g_hold{false}, g_release{false};
static void straight(const std::string &dir) {
    Run r(dir, {3 << 20, 400000, 17}, 4 << 20, 3, 1);
    REQUIRE(r.lay.n_chunks == 1);
    std::atomic<int> pieces{0};
    ckpt_stats st;
    g_before_write = [&](off_t off) {
        if (off < off_t(r.lay.header_bytes) || g_release) return;
        if (pieces++ == 0) REQUIRE(comes_true([&] { return ckpt_get_stats(r.ctx, 2, &st) == CKPT_OK && st.host_submit_ms >= 0; }));
    };
    r.snapshot(1);
    REQUIRE(ckpt_wait_immutable_window_end(r.ctx, r.compute, 1) == CKPT_OK);
    g_compute = r.compute;
    g_hold = true;
    g_emu_submit_hook = [](hipStream_t s) {
        if (s && s != g_compute && g_hold.exchange(false)) s->push([] { comes_true([] { return g_release.load(); }); });
    };
    r.snapshot(2);
    ckpt_stats first;
    const bool committed = comes_true([&] { return ckpt_get_stats(r.ctx, 1, &first) == CKPT_OK && first.committed; });
    const bool held = !g_hold && ckpt_get_stats(r.ctx, 2, &st) == CKPT_OK && !st.d2h_done;
    g_release = true;
    REQUIRE(committed && held && pieces > 2);
    g_emu_submit_hook = nullptr;
    REQUIRE(ckpt_flush(r.ctx, CKPT_ITER_ALL) == CKPT_OK);
    g_before_write = nullptr;
    r.restored(1);
    r.restored(2);
}

// Two I/O threads and a last chunk of two parts, the second of two pieces, which a thread each waits for. Both have written a piece of the first
// snapshot, which tells them from the submit thread. Of an I/O thread's waits one that no write has followed is for the end of the copies.
static thread_local bool t_io = false, t_waited = false;
static std::atomic<bool> g_watch{false}, g_at_end{false}, g_said{false};
static std::atomic<int> g_waits{0};
static ckpt_ctx *g_ctx;
static bool submitted(uint64_t it) {
    ckpt_stats st;
    return ckpt_get_stats(g_ctx, it, &st) == CKPT_OK && st.host_submit_ms >= 0;
}
static void late(const std::string &dir) {
    const uint64_t piece = DSLLM_PIECE_BYTES, chunk = 8 * piece;
    Run r(dir, {chunk + 4 * piece + piece + 4096}, chunk, 8, 2, CKPT_WINDOW_PACK);       // 8 pieces, then parts of 4 and of 2
    REQUIRE(r.lay.n_chunks == 2);
    g_ctx = r.ctx;
    std::atomic<int> arrived{0};
    g_before_write = [&](off_t off) {
        t_waited = false;
        if (g_watch && off == off_t(r.lay.header_bytes + chunk + 3 * piece)) comes_true([] { return g_waits >= 13; });    // the last piece goes to this thread
        if (off < off_t(r.lay.header_bytes) || t_io) return;
        t_io = true;
        arrived++;
        comes_true([&] { return arrived == 2; });
    };
    r.snapshot(5);
    REQUIRE(ckpt_wait_immutable_window_end(r.ctx, r.compute, 0) == CKPT_OK && ckpt_flush(r.ctx, 5) == CKPT_OK && arrived == 2);
    g_watch = true;
    g_emu_wait_hook = [] {
        if (!g_watch || !t_io) return;
        if (!t_waited) {                       // for a piece
            t_waited = true;
            if (++g_waits == 13) comes_true([] { return g_at_end.load(); });        // the last but one
            return;
        }
        g_at_end = true;                       // for the end of the copies
        g_watch = false;
        for (int i = 0; i < 300 && !submitted(2); i++) std::this_thread::sleep_for(std::chrono::milliseconds(1));
        g_said = submitted(2);
    };
    g_compute = r.compute;
    g_emu_copy_hook = [](const void *, size_t n, hipMemcpyKind kind, bool starts) {      // the last part lands when both wait for it
        if (kind == hipMemcpyDeviceToHost && starts && n == DSLLM_PIECE_BYTES + 4096) comes_true([] { return g_waits >= 14; });
    };
    r.snapshot(1);
    REQUIRE(ckpt_wait_immutable_window_end(r.ctx, r.compute, 1) == CKPT_OK && comes_true([] { return submitted(1); }));
    g_hold = true;                             // the next snapshot's first stream
    g_emu_submit_hook = [](hipStream_t s) {
        if (s && s != g_compute && g_hold.exchange(false)) s->push([] { comes_true([] { return g_release.load(); }); });
    };
    r.snapshot(2);
    ckpt_stats first;
    const bool committed = comes_true([&] { return ckpt_get_stats(r.ctx, 1, &first) == CKPT_OK && first.committed; });
    g_release = true;
    REQUIRE(g_at_end && committed && !g_said);
    g_emu_submit_hook = nullptr;
    REQUIRE(ckpt_flush(r.ctx, CKPT_ITER_ALL) == CKPT_OK);
    g_emu_wait_hook = nullptr;
    g_emu_copy_hook = nullptr;
    g_before_write = nullptr;
    r.restored(1);
    r.restored(2);
}

int main(int argc, char **argv) {
    if (argc < 3) return 2;
    const std::string dir = argv[1], what = argv[2];
    if (what == "end") end_of_copies(dir);
    else if (what == "restore" && argc > 4) restore(dir, strtoull(argv[3], nullptr, 10), strtoull(argv[4], nullptr, 10));
    else if (what == "events") events(dir);
    else if (what == "straight") straight(dir);
    else if (what == "late") late(dir);
    else if (what == "one" && argc > 3) one_chunk(dir, strtoull(argv[3], nullptr, 10));
    else return 2;
    printf("ok %s\n", what.c_str());
    return 0;
}
