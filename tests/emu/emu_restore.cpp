// Restores that a caller's stream reaches late, on the CPU model of streams and events (hip/hip_runtime.h). What work the
// caller enqueues between two restores reads must be the first one's file, whatever the second one has done to the
// context's staging memory meanwhile; and a restore that fails in the middle of its file has written its last byte when it
// returns. Meant for -fsanitize=thread and -fsanitize=address.
//   emu_restore <dir> order|failed <reduce> <direct_min>
#include <atomic>
#include <chrono>
#include <cstdio>
#include <cstdlib>
#include <string>
#include <thread>
#include <vector>

#include <sys/uio.h>
#include <unistd.h>

#include "../../include/ckpt.h"
#include "hip/hip_runtime.h"

thread_local dim3 threadIdx, blockIdx, blockDim, gridDim;
ssize_t emu_pwrite(int fd, const void *buf, size_t n, off_t off) {
    struct iovec iov = {const_cast<void *>(buf), n};
    return pwritev(fd, &iov, 1, off);
}
#define REQUIRE(x) do { if (!(x)) { printf("FAILED line %d: %s (%s)\n", __LINE__, #x, ckpt_last_error()); exit(1); } } while (0)

static const int kParams = 5;
static const uint64_t kNumel[kParams] = {3, 8193, 40000, 1000, 30001};

// per parameter a bf16 copy (its f32 tensor's upper halves: the rounding of values whose lower halves are zero) and the f32 tensor
struct State {
    std::vector<std::vector<uint8_t>> t;
    State() { for (uint64_t n : kNumel) { t.emplace_back(2 * n + 16); t.emplace_back(4 * n + 16); } }
    void fill(int it, bool pairs_hold) {
        for (int k = 0; k < kParams; k++)
            for (uint64_t e = 0; e < kNumel[k]; e++) {
                const uint16_t b = uint16_t(e * 2654435761ull + uint64_t(it) * 40503 + uint64_t(k) * 77) & 0x3FFF;
                const uint32_t u = uint32_t(b) << 16;
                memcpy(&t[2 * k][2 * e], &b, 2);
                memcpy(&t[2 * k + 1][4 * e], &u, 4);
            }
        if (!pairs_hold) t[0][0] ^= 1;
    }
};

struct Run {
    State state;
    std::vector<std::string> names;
    std::vector<int64_t> shapes;
    std::vector<ckpt_tensor_desc> descs;
    ckpt_ctx *ctx = nullptr;
    hipStream_t compute;

    Run(const std::string &dir, bool reduce, uint64_t direct_min) : shapes(2 * kParams) {
        for (int j = 0; j < 2 * kParams; j++) { names.push_back("t" + std::to_string(j)); shapes[j] = int64_t(kNumel[j / 2]); }
        for (int j = 0; j < 2 * kParams; j++) {
            ckpt_tensor_desc d{};
            d.name = names[j].c_str(); d.dtype = j % 2 ? CKPT_F32 : CKPT_BF16; d.ndim = 1; d.shape = &shapes[j]; d.dev_ptr = state.t[j].data();
            d.nbytes = (j % 2 ? 4 : 2) * kNumel[j / 2];
            descs.push_back(d);
        }
        ckpt_config cfg{};
        cfg.out_dir = dir.c_str();
        cfg.host_ring_bytes = 128 << 10;
        cfg.dma_chunk_bytes = 64 << 10;
        cfg.pack_superchunk_bytes = 128 << 10;
        cfg.n_dma_streams = 2;
        cfg.n_io_threads = 3;
        cfg.direct_min_bytes = direct_min;
        REQUIRE(ckpt_init(&cfg, &ctx) == CKPT_OK);
        if (reduce) {
            std::vector<uint32_t> derived, source;
            for (uint32_t k = 0; k < kParams; k++) { derived.push_back(2 * k); source.push_back(2 * k + 1); }
            REQUIRE(ckpt_declare_derived(ctx, derived.data(), source.data(), kParams) == CKPT_OK);
        }
        REQUIRE(ckpt_register_tensors(ctx, descs.data(), descs.size()) == CKPT_OK);
        hipStreamCreateWithFlags(&compute, hipStreamNonBlocking);
    }
    std::string snapshot(int it, bool pairs_hold) {
        emu_submit(compute, [this, it, pairs_hold] { state.fill(it, pairs_hold); });
        REQUIRE(ckpt_snapshot_async(ctx, uint64_t(it), compute) == CKPT_OK);
        REQUIRE(ckpt_wait_immutable_window_end(ctx, compute, 0) == CKPT_OK);
        REQUIRE(ckpt_flush(ctx, uint64_t(it)) == CKPT_OK);
        char name[4096];
        REQUIRE(ckpt_file_name(ctx, uint64_t(it), name, sizeof name) == CKPT_OK);
        return name;
    }
    void busy() { emu_submit(compute, [] { std::this_thread::sleep_for(std::chrono::milliseconds(200)); }); }
    ~Run() {
        REQUIRE(ckpt_destroy(ctx) == CKPT_OK);
        hipStreamDestroy(compute);
    }
};

static void order(const std::string &dir, bool reduce, uint64_t direct_min) {
    Run r(dir, reduce, direct_min);
    std::vector<std::string> file;
    std::vector<State> want(3), seen(3);
    for (int it = 0; it < 3; it++) {
        want[it].fill(it, it != 1);      // the second snapshot is a version-1 file also where pairs are declared
        file.push_back(r.snapshot(it, it != 1));
        ckpt_stats st;
        REQUIRE(ckpt_get_stats(r.ctx, uint64_t(it), &st) == CKPT_OK && st.format_version == (reduce && it != 1 ? 2 : 1));
    }
    emu_submit(r.compute, [&r] { for (auto &t : r.state.t) std::fill(t.begin(), t.end(), 0xA5); });
    r.busy();
    for (int it = 0; it < 3; it++) {
        uint64_t got = 99;
        REQUIRE(ckpt_restore(r.ctx, file[it].c_str(), r.compute, &got) == CKPT_OK && got == uint64_t(it));
        emu_submit(r.compute, [&r, &seen, it] { seen[it] = r.state; });
    }
    hipStreamSynchronize(r.compute);
    for (int it = 0; it < 3; it++)
        for (int j = 0; j < 2 * kParams; j++) {
            if (memcmp(seen[it].t[j].data(), want[it].t[j].data(), r.descs[j].nbytes) != 0) { printf("FAILED restore %d, tensor %d\n", it, j); exit(1); }
            for (uint64_t i = r.descs[j].nbytes; i < seen[it].t[j].size(); i++) REQUIRE(seen[it].t[j][i] == 0xA5);
        }
}

// The file ends two chunks after its header by the time its data is read: the first chunk's scatter kernel is queued behind
// the caller's stream when the read of a later one fails. From the return on the tensors' memory is the caller's again.
static std::string g_cut_file;
static off_t g_cut_at;
static std::atomic<bool> g_cut{false};

static void failed(const std::string &dir, bool reduce, uint64_t direct_min) {
    Run r(dir, reduce, direct_min);
    State want;
    want.fill(2, true);
    g_cut_file = r.snapshot(1, true);
    const std::string whole = r.snapshot(2, true);
    ckpt_layout lay;
    REQUIRE(ckpt_get_layout(r.ctx, &lay) == CKPT_OK);
    g_cut_at = off_t((reduce ? lay.reduced_header_bytes : lay.header_bytes) + (128 << 10));
    r.busy();
    g_cut = true;       // at the restore's first submission: it has looked at the header and the file's size by then
    g_emu_submit_hook = [](hipStream_t) { if (g_cut.exchange(false)) REQUIRE(truncate(g_cut_file.c_str(), g_cut_at) == 0); };
    REQUIRE(ckpt_restore(r.ctx, g_cut_file.c_str(), r.compute, nullptr) == CKPT_EIO);
    g_emu_submit_hook = nullptr;
    for (auto &t : r.state.t) std::fill(t.begin(), t.end(), 0x77);
    hipStreamSynchronize(r.compute);
    std::this_thread::sleep_for(std::chrono::milliseconds(100));
    for (auto &t : r.state.t) for (uint8_t b : t) REQUIRE(b == 0x77);
    REQUIRE(ckpt_restore(r.ctx, whole.c_str(), r.compute, nullptr) == CKPT_OK);      // and the context goes on working
    hipStreamSynchronize(r.compute);
    for (int j = 0; j < 2 * kParams; j++) REQUIRE(memcmp(r.state.t[j].data(), want.t[j].data(), r.descs[j].nbytes) == 0);
}

int main(int argc, char **argv) {
    if (argc < 5) return 2;
    const std::string dir = argv[1], what = argv[2];
    if (what == "order") order(dir, atoi(argv[3]) != 0, strtoull(argv[4], nullptr, 10));
    else if (what == "failed") failed(dir, atoi(argv[3]) != 0, strtoull(argv[4], nullptr, 10));
    else return 2;
    printf("ok %s\n", what.c_str());
    return 0;
}
