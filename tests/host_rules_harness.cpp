// Host-only driver of the launch rules and tables that the GPU entry points build on the host.
// argv[1] names the check; exit status 0 = it holds, 1 = it does not (with a line that says where).
#include <cstdio>
#include <cstring>

#include "../paper_1711_01912_amd/csrc/launch.hpp"

using namespace cpeval;

// The launch that clears CP leaves no thread more than its share of the batch.
static int prepare() {
    for (int32_t words : {1, 6, 300, 448})
        for (int64_t cells : {0ll, 1ll, 256ll, 257ll, 65536ll, 500000ll, 2000000ll, 0x7fffffffll}) {
            const int64_t threads = 256 * (int64_t)prepare_blocks(words, (int32_t)cells);
            const int64_t each = (cells + threads - 1) / threads;
            if (threads < words || each > std::max<int64_t>(1, (cells + 256 * 2048 - 1) / (256 * 2048))) {
                std::printf("words %d cells %lld: %lld threads\n", words, (long long)cells, (long long)threads);
                return 1;
            }
        }
    return 0;
}

int main(int argc, char **argv) {
    if (argc < 2) return 2;
    if (!std::strcmp(argv[1], "prepare")) return prepare();
    return 2;
}
