// Prints how a forward call tiles its GEMMs on 256 compute units: for every line "R C I saved" of the standard input
// "<gate/up> <down>", each "full+mi" (rows of 256-row tiles, then tiles of 32 mi rows; streamk.hpp), with "s<splits>:" before
// that of the down GEMM, or the name of the path that it takes instead.
#include <cstdio>
#include <string>
#include "../../paper_2503_21817_amd/csrc/layout.hpp"
using namespace skipffn;

static std::string rows(long R, int columns, int slabs, bool even, bool two_parts) {
    const int tiles = (int)((R + 127) / 128 * columns + 7) / 8 * 8;
    const StreamRows p = stream_rows_plan((int)R, columns, slabs, tiles < 256 ? tiles : 256, even, two_parts);
    return std::to_string(p.full) + "+" + std::to_string(p.mi);
}

int main() {
    long R, C, I;
    int saved;
    while (scanf("%ld %ld %ld %d", &R, &C, &I, &saved) == 4) {
        const ForwardPlan p = plan_forward(R, C, I, saved != 0, false, 256);
        std::string g = "few", d = "few";
        if (p.gate_up == FWD_MID) g = "mid";
        if (p.gate_up == FWD_CORE) g = rows(R, (int)((I + 127) / 128), (int)((C + 63) / 64), saved != 0, true);
        if (p.down == FWD_MID) d = "mid";
        if (p.down == FWD_CORE && p.k_down.sk_nbg > 0) d = "balanced";
        if (p.down == FWD_CORE && p.k_down.sk_nbg == 0) {
            const int s = p.k_down.splits, kt = (int)((I + 63) / 64);
            d = "s" + std::to_string(s) + ":" + rows(R, (int)((C + 255) / 256) * s, (kt + s - 1) / s, false, false);
        }
        printf("%s %s\n", g.c_str(), d.c_str());
    }
    return 0;
}
