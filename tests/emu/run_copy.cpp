// Runs the copy kernel on the CPU (tests/emu/hip/hip_runtime.h): arrays of the given byte
// sizes, each a block of exactly its size, copied in one launch and compared; built with a
// sanitizer, so an access past an array's end or two threads storing one word end the run.
// Test infrastructure.
//
// usage: run_copy to_host bytes...   (1 to MAX_COPIES even sizes)
#include "../../paper_2004_04334_amd/csrc/pxcl_kernels.hip"

#include <algorithm>
#include <cstdlib>
#include <random>

using namespace pxcl;

int main(int argc, char** argv) {
    const u32 n = u32(argc - 2);
    if (argc < 3 || n > MAX_COPIES) return 2;
    CopyArgs c{};
    std::mt19937 rng(5);
    size_t words = 0;
    u8 *src[MAX_COPIES], *dst[MAX_COPIES];
    size_t bytes[MAX_COPIES];
    for (u32 i = 0; i < n; ++i) {
        bytes[i] = strtoul(argv[2 + i], nullptr, 10);
        src[i] = static_cast<u8*>(malloc(bytes[i]));       // 16-byte aligned, as pinned and device memory
        dst[i] = static_cast<u8*>(malloc(bytes[i]));
        for (size_t j = 0; j < bytes[i]; ++j) {
            src[i][j] = u8(rng());
            dst[i][j] = u8(~src[i][j]);
        }
        c.src[i] = reinterpret_cast<const u64*>(src[i]);
        c.dst[i] = reinterpret_cast<u64*>(dst[i]);
        c.first[i] = u32(words);
        c.tail[i] = u32(bytes[i] % 8 / 2);
        words += bytes[i] / 8;
    }
    c.n = n;
    c.first[n] = u32(words);
    if (launch_copy(c, atoi(argv[1]) != 0, nullptr) != hipSuccess) return 3;
    for (u32 i = 0; i < n; ++i) {
        if (memcmp(src[i], dst[i], bytes[i]) != 0) {
            fprintf(stderr, "array %u of %zu bytes differs\n", i, bytes[i]);
            return 4;
        }
        free(src[i]);
        free(dst[i]);
    }
    return 0;
}
