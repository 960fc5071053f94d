// Host-side driver of the page backing of output arrays (test infrastructure).
#include "../../paper_1606_02862_amd/csrc/page_touch.hpp"

extern "C" int pth_touch(char* const* p, const size_t* n)
{
    std::array<std::pair<char*, size_t>, 9> spans;
    for (int i = 0; i < 9; ++i) spans[i] = {p[i], n[i]};
    pic::PageToucher t;
    t.start(spans);
    const int used = (int)t.threads.size();
    t.join();
    return used;
}
