// A shard small enough to be packed straight into its ring slot, on the CPU model of streams and events
// (hip/hip_runtime.h): the update mutates every byte right behind each window while earlier files are still being written,
// with a ring of two slots, under both window policies; every file must hold the state at its boundary, and a restore
// must bring it back. Meant for -fsanitize=thread and -fsanitize=address.
#include <cstdio>
#include <cstdlib>
#include <string>
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

int main(int argc, char **argv) {
    const std::string dir = argv[1];
    const int policy = atoi(argv[2]);
    const uint64_t sizes[] = {1, 4095, 4096, 40000, 17, 100001, 32768, 3};
    std::vector<std::vector<uint8_t>> bufs;
    std::vector<ckpt_tensor_desc> descs;
    std::vector<std::string> names;
    std::vector<int64_t> shapes(8);
    for (int k = 0; k < 8; k++) { bufs.emplace_back(sizes[k] + 32, uint8_t(k)); names.push_back("t" + std::to_string(k)); shapes[k] = int64_t(sizes[k]); }
    for (int k = 0; k < 8; k++) {
        ckpt_tensor_desc d{};
        d.name = names[k].c_str(); d.dtype = CKPT_U8; d.ndim = 1; d.shape = &shapes[k]; d.dev_ptr = bufs[k].data() + 16 + k % 3; d.nbytes = sizes[k];
        descs.push_back(d);
    }
    ckpt_config cfg{};
    cfg.out_dir = dir.c_str();
    cfg.host_ring_bytes = 1 << 20;
    cfg.dma_chunk_bytes = 512 << 10;
    cfg.pack_superchunk_bytes = 512 << 10;
    cfg.n_io_threads = 3;
    cfg.window_policy = policy;
    cfg.io_mode = CKPT_IO_MMAP;
    ckpt_ctx *ctx = nullptr;
    REQUIRE(ckpt_init(&cfg, &ctx) == CKPT_OK);
    REQUIRE(ckpt_register_tensors(ctx, descs.data(), descs.size()) == CKPT_OK);
    ckpt_layout lay;
    REQUIRE(ckpt_get_layout(ctx, &lay) == CKPT_OK && lay.n_chunks == 1);
    hipStream_t compute;
    hipStreamCreateWithFlags(&compute, hipStreamNonBlocking);
    auto value = [](int it, int k, uint64_t i) { return uint8_t(it * 37 + k * 11 + i); };
    for (int it = 1; it <= 10; it++) {
        REQUIRE(ckpt_wait_immutable_window_end(ctx, compute, 0) == CKPT_OK);
        emu_submit(compute, [&, it] { for (int k = 0; k < 8; k++) for (uint64_t i = 0; i < sizes[k]; i++) static_cast<uint8_t *>(descs[k].dev_ptr)[i] = value(it, k, i); });
        REQUIRE(ckpt_snapshot_async(ctx, uint64_t(it), compute) == CKPT_OK);
    }
    REQUIRE(ckpt_flush(ctx, CKPT_ITER_ALL) == CKPT_OK);
    char name[4096];
    for (int it = 1; it <= 10; it++) {
        REQUIRE(ckpt_file_name(ctx, uint64_t(it), name, sizeof name) == CKPT_OK);
        std::vector<uint8_t> got(lay.file_bytes), want(lay.data_bytes, 0);
        FILE *f = fopen(name, "rb");
        REQUIRE(f && fread(got.data(), 1, got.size(), f) == got.size() && fgetc(f) == EOF);
        fclose(f);
        uint64_t off = 0;
        for (int k = 0; k < 8; k++) { for (uint64_t i = 0; i < sizes[k]; i++) want[off + i] = value(it, k, i); off += (sizes[k] + 4095) / 4096 * 4096; }
        REQUIRE(memcmp(got.data() + lay.header_bytes, want.data(), want.size()) == 0);
        ckpt_stats st;
        REQUIRE(ckpt_get_stats(ctx, uint64_t(it), &st) == CKPT_OK && st.d2h_done && st.committed && st.pack_launches == 1);
    }
    REQUIRE(ckpt_file_name(ctx, 4, name, sizeof name) == CKPT_OK);
    REQUIRE(ckpt_restore(ctx, name, compute, nullptr) == CKPT_OK);
    hipStreamSynchronize(compute);
    for (int k = 0; k < 8; k++) for (uint64_t i = 0; i < sizes[k]; i++) REQUIRE(static_cast<uint8_t *>(descs[k].dev_ptr)[i] == value(4, k, i));
    REQUIRE(ckpt_destroy(ctx) == CKPT_OK);
    hipStreamDestroy(compute);
    printf("ok straight policy %d\n", policy);
    return 0;
}
