// The pack time a snapshot reports, on the CPU model of streams and events (hip/hip_runtime.h): the first super-chunk goes in
// two launches, and what passes between them is nobody's work.
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

static std::atomic<hipStream_t> g_compute{nullptr}, g_pack{nullptr};
static std::atomic<int> g_submissions{-1};

int main(int, char **argv) {
    const std::string dir = argv[1];
    std::vector<uint8_t> data(200000, 3);
    int64_t shape = int64_t(data.size());
    ckpt_tensor_desc d{};
    d.name = "t"; d.dtype = CKPT_U8; d.ndim = 1; d.shape = &shape; d.dev_ptr = data.data(); d.nbytes = data.size();
    ckpt_config cfg{};
    cfg.out_dir = dir.c_str();
    cfg.host_ring_bytes = 256 << 10;
    cfg.dma_chunk_bytes = 64 << 10;
    cfg.pack_superchunk_bytes = 256 << 10;
    ckpt_ctx *ctx = nullptr;
    REQUIRE(ckpt_init(&cfg, &ctx) == CKPT_OK);
    REQUIRE(ckpt_register_tensors(ctx, &d, 1) == CKPT_OK);
    hipStream_t compute;
    hipStreamCreateWithFlags(&compute, hipStreamNonBlocking);
    g_compute = compute;
    // The submit thread is held up for 600 ms before the fifth thing it puts on the pack stream (the first stream it uses): the wait for
    // the boundary, the first launch's start, the kernel and whatever follows the kernel come before that, the second kernel after it.
    g_emu_submit_hook = [](hipStream_t s) {
        if (g_submissions < 0 || s == g_compute) return;
        hipStream_t none = nullptr;
        g_pack.compare_exchange_strong(none, s);
        if (s == g_pack && ++g_submissions == 5) std::this_thread::sleep_for(std::chrono::milliseconds(600));
    };
    g_submissions = 0;
    REQUIRE(ckpt_snapshot_async(ctx, 1, compute) == CKPT_OK);
    REQUIRE(ckpt_wait_immutable_window_end(ctx, compute, 0) == CKPT_OK);
    REQUIRE(ckpt_flush(ctx, 1) == CKPT_OK);
    g_emu_submit_hook = nullptr;
    ckpt_stats st;
    REQUIRE(ckpt_get_stats(ctx, 1, &st) == CKPT_OK && st.pack_launches == 1 && st.d2h_done && st.committed);
    REQUIRE(st.request_to_pack_end_ms >= 600 && st.pack_ms_sum > 0);
    if (st.pack_ms_sum >= 300) { printf("FAILED pack_ms_sum %.1f of %.1f ms to the end of the packing\n", st.pack_ms_sum, st.request_to_pack_end_ms); return 1; }
    REQUIRE(ckpt_destroy(ctx) == CKPT_OK);
    hipStreamDestroy(compute);
    printf("ok pack time\n");
    return 0;
}
