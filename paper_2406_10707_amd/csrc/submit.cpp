// The submit thread: enqueues a snapshot's pack launches and device-to-host copies, and blocks on
// ring back-pressure so that the caller never does.
#include "engine_internal.hpp"

using namespace dsllm;

// A data region this small is packed straight into its ring slot over the link: the copy engine's start and the event
// between kernel and copy cost more than they bring. Request to committed file, staged -> straight: 64 KiB 116 -> 88 us,
// 1 MiB 156 -> 135, 4 MiB 316 -> 296, 8 MiB 400 -> 385, 16 MiB 586 -> 593 (with neither's file written in parts; the kernel's stores reach the copy engines'
// rate but hold compute units meanwhile, so the line is drawn where the gain is still several per cent). Not under
// policy PACK, whose window closes with the pack kernel: writing to device memory ends sooner.
constexpr uint64_t kStraightBytes = 4ull << 20;
static bool packs_straight_into_ring(const Plan &p, int policy) {
    return policy == CKPT_WINDOW_D2H && p.n_chunks == 1 && p.data_bytes <= kStraightBytes && p.segs.size() == 1 && p.segs[0].kind == CKPT_SEG_STAGED;
}

// The tiles of a snapshot's first chunk go in a launch of their own where at least so many are left behind them in the super-chunk
// (32 MiB of whole tiles): the link then starts when the first chunk is in staging and not when the whole super-chunk is
// (0.18 ms per GiB of aligned tensors, twice that beside a GEMM). The second launch and its events cost the snapshot
// 10 to 20 us: window of a 20 MiB shard in chunks of 4 MiB 540 us apart, 531 together; 60 MiB 1374, 1381; 250 MiB (chunks of
// 16 MiB) 4895, 4970.
#ifndef DSLLM_HEAD_APART_TILES
#define DSLLM_HEAD_APART_TILES 1024
#endif

static void submit_one(ckpt_ctx *c, const std::shared_ptr<Snap> &sp) {
    Snap *s = sp.get();
    const uint64_t CH = c->cfg.dma_chunk_bytes, SC = c->cfg.pack_superchunk_bytes;
    const size_t nk = c->dma.size();
    auto hip_fail = [&](const char *what, hipError_t e) { c->fail_snapshot(s, CKPT_EHIP, std::string(what) + ": " + hipGetErrorString(e)); };
    hipError_t e;
    double tier2_wait_ms = 0;

    // one snapshot's copies at a time: the previous one's last copy is over before this one's
    // boundary on the device timeline anyway (the caller closed its window), so this costs nothing there
    if (c->prev_job) {
        for (size_t k = 0; k < c->tails(c->prev_job.get()); k++) if ((e = hipEventSynchronize(c->tail(c->prev_job.get(), k))) != hipSuccess) hip_fail("tail sync", e);
        std::unique_lock<std::mutex> lk(c->mu);
        // with retention the previous commit is also what retires an older file into the spare pool this
        // snapshot is about to draw from: wait for it (it follows the last copy by one chunk write)
        c->cv_state.wait(lk, [&] { return c->prev_job->d2h_done && c->prev_job->at_tails == 0 && (c->cfg.keep_last == 0 || c->prev_job->committed); });
        // a second tier that must receive every snapshot: the previous one has to be on its way there before
        // this one may start (at most one file waits for the slower tier while another is being copied);
        // this is where a slow tier holds training back, through the window wait
        if (c->tier2_on && c->tier2_mode == CKPT_TIER2_EVERY) {
            auto w0 = Clock::now();
            c->cv_state.wait(lk, [&] { return c->prev_job->committed && !c->tier2_waiting; });
            tier2_wait_ms = ms_between(w0, Clock::now());
        }
    }

    // Everything below comes after the boundary on the device timeline. This thread first waits, on the host, until
    // the device has reached the boundary, and only then enqueues the snapshot's kernels and copies. A caller's
    // host thread may be whole steps ahead of its device; work enqueued at request time would sit behind an
    // unsignalled event at the head of the pack and copy queues all that while, and the command processor pays
    // for blocked queues on every dispatch of the caller's own stream: measured, 12 to 20 us per kernel launch, which
    // made every step between a request and its boundary 1.7 % slower (the Adam phase of the 7B workload 42.1
    // instead of 36.2 ms, its GEMM phase +1.1 %). The device-side wait below stays as the ordering guarantee.
    if ((e = hipEventSynchronize(s->ev_boundary)) != hipSuccess) hip_fail("boundary sync", e);
    if ((e = hipStreamWaitEvent(c->pack_stream, s->ev_boundary, 0)) != hipSuccess) hip_fail("wait boundary", e);

    // Data reduction: with derived tensors declared, the captured state is checked on the device first (every bf16
    // copy against the rounding of its f32 source). The verdict decides which of the registration's two plans this
    // snapshot is written with; this thread waits for it (some milliseconds after the boundary), the caller does not.
    const Plan *chosen = &c->plan;
    const ckpt_tile *chosen_tiles = c->dev_tiles;
    if (c->have_rplan) {
        bool launched = true;
        if ((e = hipEventRecord(c->ev_verify_start, c->pack_stream)) != hipSuccess) { hip_fail("record", e); launched = false; }
        if (launched && (e = launch_verify_pairs(c->dev_pairs, c->plan.n_pair_blocks, c->plan.pair_tiles.size(), c->dev_flag, c->pack_stream)) != hipSuccess) { hip_fail("verify launch", e); launched = false; }
        if (launched && (e = hipMemcpyAsync(c->host_flag, c->dev_flag, sizeof(uint32_t), hipMemcpyDeviceToHost, c->pack_stream)) != hipSuccess) { hip_fail("verdict copy", e); launched = false; }
        if (launched && (e = hipEventRecord(c->ev_verify_done, c->pack_stream)) != hipSuccess) { hip_fail("record", e); launched = false; }
        if (launched && (e = hipEventSynchronize(c->ev_verify_done)) != hipSuccess) { hip_fail("verdict sync", e); launched = false; }
        if (launched && *c->host_flag == 0) { chosen = &c->rplan; chosen_tiles = c->dev_rtiles; }   // anything else: the full file
        float vms = 0;
        if (launched && hipEventElapsedTime(&vms, c->ev_verify_start, c->ev_verify_done) == hipSuccess) s->verify_ms = vms;
    }
    const Plan &p = *chosen;
    s->chunks_left = p.n_chunks;
    {
        std::lock_guard<std::mutex> lk(c->mu);
        s->plan = chosen;
        s->dev_tiles = chosen_tiles;
    }

    // file and header
    const bool use_mmap = c->cfg.io_mode == CKPT_IO_MMAP;
    memcpy(c->hdr_buf, p.header.data(), p.header_bytes);
    for (int i = 0; i < 8; i++) c->hdr_buf[16 + i] = uint8_t(s->iter >> (8 * i));
    FileSlot reuse;
    std::vector<FileSlot> wrong_size;
    {
        std::lock_guard<std::mutex> lk(c->mu);
        while (!c->spares.empty() && reuse.fd < 0) {
            FileSlot f = c->spares.back();
            c->spares.pop_back();
            if (f.bytes == p.file_bytes()) reuse = f; else wrong_size.push_back(f);
        }
    }
    // a spare of another size (the previous snapshot had the other format version) cannot be overwritten in place
    for (auto &f : wrong_size) { f.close_all(); unlink(f.path.c_str()); }
    std::string ferr;
    if (reuse.fd >= 0) {
        // a retired file of this registration: same size, pages allocated, still open (and mapped);
        // every byte of it is rewritten (header, data and padding), so nothing is truncated
        s->tmp_path = reuse.path;
        s->fd = reuse.fd;
        s->map = reuse.map;
    } else {
        int flags = (use_mmap ? O_RDWR : O_WRONLY) | O_CREAT | O_TRUNC | (c->cfg.o_direct ? O_DIRECT : 0);
        s->fd = open(s->tmp_path.c_str(), flags, 0644);
        if (s->fd < 0) ferr = std::string("open: ") + strerror(errno);
        else if (use_mmap) {
            // stores into a mapping cannot report "no space left" as an error code: check the room first
            struct statvfs vfs;
            if (fstatvfs(s->fd, &vfs) == 0 && uint64_t(vfs.f_bavail) * vfs.f_frsize < p.file_bytes()) ferr = "not enough free space for the checkpoint file";
            else if (ftruncate(s->fd, off_t(p.file_bytes())) != 0) ferr = std::string("ftruncate: ") + strerror(errno);
            else {
                void *m = mmap(nullptr, p.file_bytes(), PROT_READ | PROT_WRITE, MAP_SHARED, s->fd, 0);
                if (m == MAP_FAILED) ferr = std::string("mmap: ") + strerror(errno);
                else s->map = static_cast<uint8_t *>(m);
            }
        }
    }
    if (ferr.empty() && s->fd >= 0) {
        if (s->map) memcpy(s->map, c->hdr_buf, p.header_bytes);
        else if (!pwrite_all(s->fd, c->hdr_buf, p.header_bytes, 0, &ferr)) {}
    }
    if (!ferr.empty()) {
        c->fail_snapshot(s, CKPT_EIO, s->tmp_path + ": " + ferr);
        if (s->map) munmap(s->map, p.file_bytes());
        if (s->fd >= 0) { close(s->fd); unlink(s->tmp_path.c_str()); }
        s->map = nullptr; s->fd = -1;
    }

    double bp_ms = 0;
    auto take_slot = [&]() -> uint64_t {      // the next ring slot; waits until it has been written to its file
        const uint64_t slot = c->ring_next++ % c->n_slots;
        std::unique_lock<std::mutex> lk(c->mu);
        if (c->slot_state[slot] != SLOT_FREE) {
            auto w0 = Clock::now();
            c->cv_state.wait(lk, [&] { return c->slot_state[slot] == SLOT_FREE; });
            bp_ms += ms_between(w0, Clock::now());
        }
        c->slot_state[slot] = SLOT_BUSY;
        return slot;
    };
    // Chunk ch goes to the file in pieces of at most piece_bytes. Its arrival in `slot` is the event `whole`, or part by part of part_bytes
    // those in `parts`. A piece ends where its part does: it waits for one event.
    auto hand_to_io = [&](uint64_t ch, uint64_t slot, uint64_t piece_bytes, hipEvent_t whole, uint64_t part_bytes = 0, const hipEvent_t *parts = nullptr) {
        const uint64_t nbytes = p.chunk_bytes(ch);
        uint32_t n_pieces = 0;
        {
            std::lock_guard<std::mutex> lk(c->mu);
            for (uint64_t at = 0; at < nbytes; n_pieces++) {
                const uint64_t part = parts ? at / part_bytes : 0;
                IoJob job;
                job.kind = IoJob::WRITE;
                job.snap = sp;
                job.slot = slot;
                job.slot_off = at;
                job.file_off = p.header_bytes + ch * CH + at;
                job.nbytes = std::min(piece_bytes, (parts ? std::min(nbytes, (part + 1) * part_bytes) : nbytes) - at);
                job.landed = parts ? parts[part] : whole;
                at += job.nbytes;
                job.last = ch + 1 == p.n_chunks && (parts ? at == nbytes : job.slot_off == 0);
                job.ends = ch + 1 == p.n_chunks && (parts || job.last);
                c->io_q.push_back(std::move(job));
            }
            c->slot_pieces_left[slot] = n_pieces;
        }
        if (n_pieces == 1) c->cv_io.notify_one();
        else c->cv_io.notify_all();
    };
    auto all_submitted = [&] {
        std::vector<uint8_t>().swap(s->host_capture);   // every byte of it is in a ring slot by now
        std::lock_guard<std::mutex> lk(c->mu);
        s->backpressure_ms = bp_ms + tier2_wait_ms;
        s->t_submitted = Clock::now();
        s->packs_submitted = s->submitted = true;
        c->prev_job = sp;
        c->cv_state.notify_all();
    };

    if (packs_straight_into_ring(p, s->policy)) {
        // The pack kernel writes the ring slot itself: one launch instead of a launch, an event and a copy behind it. One event behind it
        // stands for the arrival in the slot, the end of the packing and the ends of the copies. With an event for each, and one in front of
        // the kernel, the last of them was there 48 us after the first for a kernel of 15 us, now 19 us after its start:
        // request to committed file 0.46 MB 129..137 -> 110..114 us, 0.5 MB 123..140 -> 105..122, 1.7 MB 140..154 -> 136..148, 3.4 MB even.
        const uint64_t slot = take_slot();
        s->straight = true;
        s->straight_slot = slot;
        if ((e = launch_pack(s->dev_tiles, p.tiles.size(), c->ring + slot * CH, 0, c->pack_stream, c->ev_pack_start[0], c->ev_pack_end[0])) != hipSuccess)
            hip_fail("pack launch", e);
        if ((e = hipEventRecord(c->ev_slot[slot], c->pack_stream)) != hipSuccess) hip_fail("record", e);
        hand_to_io(0, slot, even_piece_bytes(p.data_bytes, uint64_t(c->cfg.n_io_threads)), c->ev_slot[slot]);
        all_submitted();
        return;
    }

    if (p.n_direct)   // these copies read the tensors themselves
        for (size_t k = 0; k < nk; k++)
            if ((e = hipStreamWaitEvent(c->dma[k], s->ev_boundary, 0)) != hipSuccess) hip_fail("wait boundary", e);
    // Pack launches run ahead of the copies: as far as staging allows when the window closes with the last pack
    // (policy PACK: get the reads of the tensors over with), `ahead` = two staging slots otherwise (under the
    // paper's rule nothing is gained by packing earlier, and a burst of pack kernels would only compete with the
    // forward pass). Pack sc needs the staging slot that the copies of super-chunk sc - ahead read (ahead <= n_stage,
    // copies are in order): this thread waits for those copies on the host and launches the pack then.
    const uint64_t ahead = s->policy == CKPT_WINDOW_PACK ? c->n_stage : std::min<uint64_t>(c->n_stage, 2);
    const uint64_t behind_head = p.first_tile_at(0, CH);      // first tile that is not the first chunk's
    const bool head_apart = p.n_chunks > 1 && SC > CH && p.sc_first_tile[0] < behind_head && behind_head + DSLLM_HEAD_APART_TILES <= p.sc_first_tile[1];
    s->head_apart = head_apart;
    auto enqueue_pack = [&](uint64_t sc) {
        const uint64_t stage = sc % c->n_stage;
        if (sc >= ahead)
            for (size_t k = 0; k < nk; k++) {
                // host first (this thread sleeps until the staging slot is free), so that the pack queue never holds a
                // launch parked behind an unsignalled event while the copies run: see the boundary wait above.
                hipEvent_t freed = c->ev_stage_done[(sc - ahead) % c->n_stage][k];
                if ((e = hipEventSynchronize(freed)) != hipSuccess) hip_fail("stage sync", e);
                if ((e = hipStreamWaitEvent(c->pack_stream, freed, 0)) != hipSuccess) hip_fail("wait stage", e);
            }
        uint64_t t0 = p.sc_first_tile[sc];
        const uint64_t t1 = p.sc_first_tile[sc + 1];
        hipEvent_t start = c->ev_pack_start[sc];
        if (head_apart && sc == 0) {   // each of the two launches has its own start and end, as the pack time is the sum of the launches'
            if ((e = launch_pack(s->dev_tiles + t0, behind_head - t0, c->staging, 0, c->pack_stream, start, c->ev_head_end)) != hipSuccess) hip_fail("pack launch", e);
            if ((e = hipEventRecord(c->ev_packed_head, c->pack_stream)) != hipSuccess) hip_fail("record", e);
            t0 = behind_head;
            start = c->ev_rest_start;
        }
        if ((e = launch_pack(s->dev_tiles + t0, t1 - t0, c->staging + stage * SC, sc * SC, c->pack_stream, start, c->ev_pack_end[sc])) != hipSuccess)
            hip_fail("pack launch", e);
        if ((e = hipEventRecord(c->ev_packed[sc], c->pack_stream)) != hipSuccess) hip_fail("record", e);
        if (sc + 1 == p.n_superchunks) {   // every read of the tensors is now in the pack stream
            std::lock_guard<std::mutex> lk(c->mu);
            s->packs_submitted = true;
            c->cv_state.notify_all();
        }
    };
    // The last chunks are shared among the copy streams, part by part in turn, and written part by part. The streams otherwise
    // end with a chunk each, and the last ones land together: 1.2 ms of writing behind the last copy with two of 64 MiB, 0.3 in parts.
    // One chunk more than there are streams, so that the I/O threads have caught up when the last one lands. The events
    // are the context's: they must not be in use for the snapshot before, which a slow disk may still be writing. Not for many
    // chunks of more than 64 MiB: beside the training step every copy more costs the system runtime some 40 us (1.74 GB in chunks of
    // 256 MiB, the last three in parts: copies at 55.8 GB/s instead of 56.6), and the end is little of the whole there. In chunks of 64 MiB the
    // copies beside the step pay too, 55.3 GB/s instead of 55.9, with the same stall; alone the file is committed sooner, 0.2 GB 4.6 -> 4.1 ms,
    // 1 GB 20.0 -> 19.6 (in chunks of 256 MiB 22.0 -> 19.8), 1.7 GB 31.9 -> 31.5. Two chunks in parts cost as much as three. (Parts of
    // 2 to 16 MiB of the last chunk alone: 0.1 GB committed 6 % sooner, but a window 3 % longer.) A single chunk has a rule of its own (kOneChunkStep).
    const bool one = p.n_chunks == 1;
    const uint64_t part_bytes = one ? one_chunk_part_bytes(p.data_bytes) : kPartBytes;
    uint64_t shared = 0;             // so many of the last chunks go in parts
    if (c->shares_last_chunks() && (one ? part_bytes < p.data_bytes : CH <= 4 * kPartBytes || p.n_chunks <= 2 * (nk + 1))) {
        std::lock_guard<std::mutex> lk(c->mu);
        if (!c->prev_job || c->prev_job->committed) shared = std::min<uint64_t>(p.n_chunks, nk + 1);
    }
    const uint64_t piece_bytes = one ? even_piece_bytes(shared ? part_bytes : p.data_bytes, uint64_t(c->cfg.n_io_threads)) : kPieceBytes;
    for (uint64_t sc = 0; sc < std::min<uint64_t>(ahead, p.n_superchunks); sc++) enqueue_pack(sc);
    for (uint64_t sc = 0; sc < p.n_superchunks; sc++) {
        const uint64_t stage = sc % c->n_stage;
        uint8_t *stage_base = c->staging + stage * SC;
        auto wait_packed = [&](size_t k, hipEvent_t packed) { if ((e = hipStreamWaitEvent(c->dma[k], packed, 0)) != hipSuccess) hip_fail("wait packed", e); };
        const bool head = head_apart && sc == 0;
        bool only_head = head;       // the first copy stream has waited for the first chunk's launch alone
        if (head) wait_packed(0, c->ev_packed_head);
        for (size_t k = head ? 1 : 0; k < nk; k++) wait_packed(k, c->ev_packed[sc]);

        const uint64_t c0 = sc * (SC / CH);
        const uint64_t c1 = std::min<uint64_t>(p.n_chunks, c0 + SC / CH);
        for (uint64_t ch = c0; ch < c1; ch++) {
            const size_t k = ch % nk;
            const bool in_parts = ch + shared >= p.n_chunks;
            if (only_head && ch > 0 && (in_parts || k == 0)) { wait_packed(0, c->ev_packed[0]); only_head = false; }
            const uint64_t slot = take_slot();
            if (ch == 0 && (e = hipEventRecord(c->ev_first_copy, c->dma[k])) != hipSuccess) hip_fail("record", e);
            // the chunk's segments: packed bytes out of staging, large tensors out of their own memory,
            // the padding behind those zero-filled here (the slot belongs to this thread until the copy event)
            uint8_t *slot_base = c->ring + slot * CH;
            const hipEvent_t *parts = in_parts ? c->ev_part[p.n_chunks - 1 - ch].data() : nullptr;
            auto stream_of = [&](uint64_t part) { return c->dma[one ? k : (k + part) % nk]; };
            uint64_t part = 0;
            for (uint64_t j = p.chunk_first_seg[ch]; j < p.chunk_first_seg[ch + 1]; j++) {
                const ckpt_segment &sg = p.segs[j];
                const uint64_t at = sg.data_off - ch * CH;
                uint8_t *dst = slot_base + at;
                if (sg.kind == CKPT_SEG_ZERO) { memset(dst, 0, sg.nbytes); continue; }
                if (sg.kind == CKPT_SEG_HOST) {   // from the copy taken at the request
                    const TensorInfo &ti = p.tensors[sg.tensor];
                    memcpy(dst, s->host_capture.data() + ti.capture_off + (sg.src - ti.dev_addr), sg.nbytes);
                    continue;
                }
                const void *src = sg.kind == CKPT_SEG_DIRECT ? reinterpret_cast<const void *>(sg.src)
                                                             : static_cast<const void *>(stage_base + (sg.data_off - sc * SC));
                for (uint64_t done = 0; done < sg.nbytes;) {
                    for (; in_parts && part < (at + done) / part_bytes; part++)      // every copy of an earlier part is enqueued
                        if ((e = hipEventRecord(parts[part], stream_of(part))) != hipSuccess) hip_fail("record", e);
                    const uint64_t n = std::min(sg.nbytes - done, (in_parts ? (part + 1) * part_bytes : CH) - (at + done));
                    e = hipMemcpyAsync(dst + done, static_cast<const uint8_t *>(src) + done, n, hipMemcpyDeviceToHost, stream_of(part));
                    if (e != hipSuccess) hip_fail("hipMemcpyAsync D2H", e);
                    done += n;
                }
            }
            if (in_parts) {
                for (; part * part_bytes < p.chunk_bytes(ch); part++)
                    if ((e = hipEventRecord(parts[part], stream_of(part))) != hipSuccess) hip_fail("record", e);
            } else if ((e = hipEventRecord(c->ev_slot[slot], c->dma[k])) != hipSuccess) hip_fail("record", e);
            const bool last = ch + 1 == p.n_chunks;
            if (ch + 1 == c1)
                for (size_t kk = 0; kk < nk; kk++)
                    if ((e = hipEventRecord(c->ev_stage_done[stage][kk], c->dma[kk])) != hipSuccess) hip_fail("record", e);
            if (last)
                for (size_t kk = 0; kk < nk; kk++)
                    if ((e = hipEventRecord(c->ev_job_tail[kk], c->dma[kk])) != hipSuccess) hip_fail("record", e);
            hand_to_io(ch, slot, piece_bytes, c->ev_slot[slot], part_bytes, parts);
        }
        // The next pack launch goes out one round late, after this super-chunk's copies have been enqueued: its host-side
        // wait is for the copies of the previous super-chunk, and the copy engines have this one's to go on with. The
        // pack of super-chunk sc + 1 was launched a round ago, before the copies above that wait for it.
        if (sc >= 1 && sc - 1 + ahead < p.n_superchunks) enqueue_pack(sc - 1 + ahead);
    }
    all_submitted();
}

void dsllm::submit_thread_main(ckpt_ctx *c) {
    (void)hipSetDevice(c->device);
    for (;;) {
        std::shared_ptr<Snap> sp;
        {
            std::unique_lock<std::mutex> lk(c->mu);
            c->cv_submit.wait(lk, [&] { return c->stopping || !c->submit_q.empty(); });
            if (c->submit_q.empty()) return;
            sp = c->submit_q.front();
            c->submit_q.pop_front();
        }
        submit_one(c, sp);
    }
}

