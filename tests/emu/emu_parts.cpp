// Snapshots in parts, on the CPU model of streams and events (hip/hip_runtime.h).
//   end      a slow sink: once its copies have landed, a snapshot says so, and the next one starts, while its last chunk is
//            still being written
//   emu_parts <dir> end
#include <atomic>
#include <chrono>
#include <cstdio>
#include <cstdlib>
#include <functional>
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

    Run(const std::string &dir, const std::vector<uint64_t> &sizes, uint64_t chunk, uint64_t slots, int io_threads) {
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

int main(int argc, char **argv) {
    if (argc < 3) return 2;
    const std::string dir = argv[1], what = argv[2];
    if (what == "end") end_of_copies(dir);
    else return 2;
    printf("ok %s\n", what.c_str());
    return 0;
}
