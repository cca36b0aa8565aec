/*
 * Runs the library's encode path -- host planning and the encode kernels' own source -- on host
 * threads (hip/hip_runtime.h and l3_gfx950.h beside this file) and compares the files it writes
 * with expected ones from a case file.  "Device" buffers are heap blocks of exactly the size the
 * interface promises: an image ends with the last pixel of its last row, a file's buffer with
 * its last byte (or wherever the case says), so under AddressSanitizer any access outside them
 * ends the run; under ThreadSanitizer any two accesses to LDS, the workspace or the files that no
 * barrier orders do.
 *
 * usage: encode_cpu <case file> [sequence]      (written by tests/test_encoder_cpu_build.py)
 * sequence: what each call of the case is, one letter each: e an ordinary call; x one
 * whose files are not looked at; c a call while the
 * stream captures (only recorded); r a replay of what was recorded; p a replay of its first workgroup alone, whose
 * files are not looked at; d disturbs the words that one-kernel calls take their tickets from; l puts the
 * number of the context's launches near its end.  Without it all are ordinary.
 * Test infrastructure.
 */
#include <hip/hip_runtime.h>

#include "l3_gfx950.h"

/* the kernel source under test: the library's, unless the build names another (a copy with a
 * planted mistake, to show that the sanitizers see it) */
#ifndef L3_KERNEL_SOURCE
#define L3_KERNEL_SOURCE "../../../paper_2208_08711_amd/csrc/l3_encode.hip"
#endif
#include L3_KERNEL_SOURCE

#include <cstdio>
#include <string>

namespace {

struct Reader {
    FILE* f;
    template <class T> T get() {
        T v;
        if (std::fread(&v, sizeof v, 1, f) != 1) { std::fprintf(stderr, "case file too short\n"); std::exit(2); }
        return v;
    }
    void bytes(void* to, size_t n) {
        if (n && std::fread(to, 1, n, f) != n) { std::fprintf(stderr, "case file too short\n"); std::exit(2); }
    }
};

constexpr uint8_t kPoison = 0xA5;

}  // namespace

int main(int argc, char** argv) {
    if (argc != 2 && argc != 3) return 2;
    Reader in{std::fopen(argv[1], "rb")};
    if (!in.f) return 2;
    if (in.get<uint32_t>() != 0x4345334Cu) return 2;       /* "L3EC" */
    const int n = (int)in.get<uint32_t>(), calls = (int)in.get<uint32_t>();
    std::vector<l3_encode_item> items((size_t)n);
    std::vector<uint8_t*> images, files;
    std::vector<std::vector<uint8_t>> expected((size_t)n);
    for (int i = 0; i < n; ++i) {
        l3_encode_item& it = items[(size_t)i];
        std::memset(&it, 0, sizeof it);
        it.width = in.get<uint32_t>();
        it.height = in.get<uint32_t>();
        it.patch = (uint8_t)in.get<uint32_t>();
        const uint32_t pad = in.get<uint32_t>(), odd = in.get<uint32_t>();   /* bytes between rows, and ahead of the image */
        it.file_cap = (size_t)in.get<uint64_t>();
        it.row_stride = 3 * (size_t)it.width + pad;
        uint8_t* image = static_cast<uint8_t*>(std::malloc(odd + (it.height - 1) * it.row_stride + 3 * (size_t)it.width));
        images.push_back(image);
        it.d_rgb = image + odd;
        std::memset(image, 0xEE, odd + (it.height - 1) * it.row_stride);
        for (uint32_t y = 0; y < it.height; ++y) in.bytes(image + odd + y * it.row_stride, 3 * (size_t)it.width);
        uint8_t* file = static_cast<uint8_t*>(std::malloc(it.file_cap ? it.file_cap : 1));
        files.push_back(file);
        it.d_file = file;
        expected[(size_t)i].resize((size_t)in.get<uint64_t>());
        in.bytes(expected[(size_t)i].data(), expected[(size_t)i].size());
    }
    std::fclose(in.f);

    l3_ctx* ctx = new l3_ctx;                               /* the encoder uses its device and its own state only */
    uint64_t* lengths = static_cast<uint64_t*>(std::malloc(sizeof(uint64_t) * (size_t)n));
    uint32_t* status = static_cast<uint32_t*>(std::malloc(sizeof(uint32_t) * (size_t)n));
    int rc = 0;
    const std::string sequence = argc == 3 ? argv[2] : std::string((size_t)calls, 'e');
    l3cpu_stream captured;
    for (int call = 0; call < (int)sequence.size() && rc == 0; ++call) {   /* the workspace of the first call serves the others */
        for (int i = 0; i < n; ++i) std::memset(files[(size_t)i], kPoison, items[(size_t)i].file_cap);
        std::memset(lengths, 0xFF, sizeof(uint64_t) * (size_t)n);
        std::memset(status, 0xFF, sizeof(uint32_t) * (size_t)n);
        /* ordinary calls without and with status words in turn */
        uint32_t* const words = argc == 2 && call % 2 ? nullptr : status;
        l3_status st = L3_OK;
        captured.capturing = sequence[(size_t)call] == 'c';
        if (captured.capturing) captured.kept.clear();
        if (std::strchr("exc", sequence[(size_t)call]))
            st = l3_encode_batch(ctx, items.data(), n, lengths, words, argc == 2 ? nullptr : &captured);
        if (sequence[(size_t)call] == 'r') captured.replay();
        if (sequence[(size_t)call] == 'p') captured.replay(1);
        if (st != L3_OK) { std::fprintf(stderr, "call failed: %s\n", l3_status_string(st)); rc = 1; }
        if (sequence[(size_t)call] == 'd')
            for (int i = 0; i < n; ++i)
                for (L3Ticket& ticket : ctx->enc->d_words[i].ticket) ticket.next += 2;
        if (sequence[(size_t)call] == 'l') {
            const uint64_t next = kLastNumber - 4;
            ctx->enc->chain_number = next - 1;
            for (uint32_t i = 0; i < kMostChainImages; ++i) ctx->enc->d_words[i].ticket[next & 1].next = next << kNumberShift;
        }
        if (sequence[(size_t)call] != 'e' && sequence[(size_t)call] != 'r') continue;
        for (int i = 0; i < n && rc == 0; ++i) {
            const std::vector<uint8_t>& want = expected[(size_t)i];
            const size_t cap = items[(size_t)i].file_cap;
            const l3_encode_item& it = items[(size_t)i];
            const size_t header = 13 + 12 * (size_t)((it.width + it.patch - 1) / it.patch) * ((it.height + it.patch - 1) / it.patch);
            const bool fits = want.size() <= cap;
            if (lengths[i] != want.size()) { std::fprintf(stderr, "MISMATCH: length, image %d: %llu\n", i, (unsigned long long)lengths[i]); rc = 1; }
            if (words && status[i] != (fits ? 0u : 1u)) { std::fprintf(stderr, "MISMATCH: status, image %d: %u\n", i, status[i]); rc = 1; }
            /* without room for the whole file the header is written if it fits, nothing else */
            const size_t written = fits ? want.size() : (header <= cap ? header : 0);
            for (size_t k = 0; k < cap && rc == 0; ++k)
                if (files[(size_t)i][k] != (k < written ? want[k] : kPoison)) {
                    std::fprintf(stderr, "MISMATCH: image %d (%ux%u, N = %u), byte %zu of %zu\n", i, it.width, it.height, it.patch, k, want.size());
                    rc = 1;
                }
        }
    }
    l3_encode_state_free(ctx->enc);
    delete ctx;
    for (uint8_t* p : images) std::free(p);
    for (uint8_t* p : files) std::free(p);
    std::free(lengths);
    std::free(status);
    if (rc == 0) std::printf("ok: %d images, %d calls\n", n, (int)sequence.size());
    return rc;
}
