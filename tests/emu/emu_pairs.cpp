// Host emulation of the derivation kernels under AddressSanitizer (see hip/hip_runtime.h here): random pairs of a bf16 and an
// f32 tensor, cut into work items by the planner. Every tensor sits in a buffer of exactly its bytes, at an address aligned to
// its element size only, so an access past it is reported. The check must pass over pairs that hold and find one wrong
// element anywhere; the regeneration must write every element and nothing else. Compiled with a small
// DSLLM_PAIR_TILES_PER_LAUNCH, so that tables go in several launches.
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <string>
#include <vector>

#include "../../paper_2406_10707_amd/csrc/derive_kernels.hip"

thread_local dim3 threadIdx, blockIdx, blockDim, gridDim;
ssize_t emu_pwrite(int, const void *, size_t, off_t) { return -1; }   // no file is written here

static uint16_t rounding(uint32_t u) {
    if ((u & 0x7FFFFFFFu) > 0x7F800000u) return uint16_t((u >> 16) | 0x40u);
    return uint16_t((u + 0x7FFFu + ((u >> 16) & 1u)) >> 16);
}

int main(int argc, char **argv) {
    using namespace dsllm;
    uint64_t state = argc > 1 ? strtoull(argv[1], nullptr, 10) : 1;
    const int n = argc > 2 ? atoi(argv[2]) : 60;
    const uint64_t limit = argc > 3 ? strtoull(argv[3], nullptr, 10) : 10000;   // largest random count
    auto rnd = [&] { state = state * 6364136223846793005ull + 1442695040888963407ull; return state >> 33; };
    static const uint64_t edge[] = {1, 2, 3, 4, 5, 255, 256, 257, 259, 508, 511, 512, 513, 516, 1023, 1024, 1025, 4092, 4095, 4096, 4097, 4608, 4609, 8191, 8192, 8193};
    struct Pair { uint8_t *f32, *bf16; uint64_t count; void *base[2]; };
    std::vector<Pair> ps;
    std::vector<std::string> names;
    std::vector<int64_t> shapes(n);
    std::vector<ckpt_tensor_desc> descs;
    DerivedPairs pairs;
    for (int k = 0; k < n; k++) {
        Pair p;
        do p.count = rnd() % 2 ? edge[rnd() % 26] : 1 + rnd() % limit; while (p.count > limit);
        // the end of each buffer is the tensor's end; the start is off by some elements
        const uint64_t lead32 = 4 * (rnd() % 4), lead16 = 2 * (rnd() % 8);
        p.f32 = static_cast<uint8_t *>(p.base[0] = malloc(lead32 + 4 * p.count)) + lead32;
        p.bf16 = static_cast<uint8_t *>(p.base[1] = malloc(lead16 + 2 * p.count)) + lead16;
        for (uint64_t e = 0; e < p.count; e++) {
            uint32_t u = uint32_t(rnd() * 2654435761u);
            if (rnd() % 16 == 0) u = 0x7F800000u | (u & 0x807FFFFFu);      // infinities and NaNs
            if (rnd() % 16 == 0) u = (u & 0xFFFF0000u) | 0x8000u;         // ties
            memcpy(p.f32 + 4 * e, &u, 4);
        }
        memset(p.bf16, 0x5A, 2 * p.count);
        ps.push_back(p);
        names.push_back("p" + std::to_string(k));
        names.push_back("m" + std::to_string(k));
    }
    for (int k = 0; k < n; k++) {
        shapes[k] = int64_t(ps[k].count);
        ckpt_tensor_desc d{};
        d.ndim = 1; d.shape = &shapes[k];
        d.name = names[2 * k].c_str(); d.dtype = CKPT_BF16; d.dev_ptr = ps[k].bf16; d.nbytes = 2 * ps[k].count; descs.push_back(d);
        d.name = names[2 * k + 1].c_str(); d.dtype = CKPT_F32; d.dev_ptr = ps[k].f32; d.nbytes = 4 * ps[k].count; descs.push_back(d);
        pairs.derived.push_back(uint32_t(2 * k)); pairs.source.push_back(uint32_t(2 * k + 1));
    }
    ckpt_config cfg{};
    ResolvedConfig rc;
    Plan plan;
    std::string err;
    if (resolve_config(&cfg, &rc, &err) || build_plan(descs.data(), descs.size(), rc, &plan, &err, &pairs, true)) { printf("plan: %s\n", err.c_str()); return 2; }
    const std::vector<PairTile> &t = plan.pair_tiles;
    uint64_t elements = 0, want_elements = 0;
    for (size_t i = 0; i < t.size(); i++) {
        elements += t[i].count;
        if (t[i].count == 0 || t[i].count > kPairTileElems || (t[i].count > kPairSmallElems) != (i < plan.n_pair_blocks)) { printf("work item %zu out of place\n", i); return 1; }
    }
    for (auto &p : ps) want_elements += p.count;
    if (elements != want_elements) { printf("work items hold %llu elements\n", (unsigned long long)elements); return 1; }

    auto check = [&] {
        uint32_t *flag = static_cast<uint32_t *>(malloc(4));
        *flag = 7;
        launch_verify_pairs(t.data(), plan.n_pair_blocks, t.size(), flag, nullptr);
        const uint32_t r = *flag;
        free(flag);
        return r;
    };
    if (check() != 1) { printf("wrong copies not found\n"); return 1; }
    launch_derive_pairs(t.data(), plan.n_pair_blocks, t.size(), nullptr);
    for (int k = 0; k < n; k++)
        for (uint64_t e = 0; e < ps[k].count; e++) {
            uint32_t u; uint16_t b;
            memcpy(&u, ps[k].f32 + 4 * e, 4);
            memcpy(&b, ps[k].bf16 + 2 * e, 2);
            if (b != rounding(u)) { printf("pair %d, element %llu of %llu: not regenerated\n", k, (unsigned long long)e, (unsigned long long)ps[k].count); return 1; }
        }
    if (check() != 0) { printf("a pair that holds is refused\n"); return 1; }
    for (int k = 0; k < n; k += 1 + n / 30)
        for (uint64_t e : {uint64_t(0), ps[k].count / 2, ps[k].count - 1}) {
            ps[k].bf16[2 * e] ^= 1;
            if (check() != 1) { printf("pair %d: wrong element %llu of %llu not found\n", k, (unsigned long long)e, (unsigned long long)ps[k].count); return 1; }
            ps[k].bf16[2 * e] ^= 1;
        }
    for (auto &p : ps) { free(p.base[0]); free(p.base[1]); }
    printf("ok items %zu, of a block %llu\n", t.size(), (unsigned long long)plan.n_pair_blocks);
    return 0;
}
