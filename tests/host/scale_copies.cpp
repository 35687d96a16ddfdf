// Runs the copies of the MXFP4 tiles (csrc/scale_chunks.h, csrc/code_rows.h) on the host, lane by lane and in the order of the kernel's units, and
// checks them: what lands is what the unit needs, copies of one chunk never write one place from two, scalar offsets stay within the operand.
#include "code_rows.h"
#include "scale_chunks.h"

namespace arcq {
Host host;
}
using namespace arcq;

static long wrong = 0;      // bytes of rows of the tile that a unit found different
static long checked = 0;

static std::vector<uint8_t> operand(int rows, int nb, uint32_t seed) {
    std::vector<uint8_t> out((size_t)rows * nb);
    for (auto& b : out) b = (uint8_t)((seed = seed * 1664525u + 1013904223u) >> 24);
    return out;
}

struct Problem {
    int M, N, nb, m0, n0, u0, u1;
    std::vector<uint8_t> a, w;
};

template <typename At>
static void compare(const Problem& p, int unit, bool zero_past_row, At at) {
    for (int side = 0; side < 2; ++side) {
        const int rows = side ? p.N : p.M, first = side ? p.n0 : p.m0;
        for (int r = 0; first + r < rows && at(side, r); ++r)
            for (int b = 0; b < 8; ++b) {
                if (8 * unit + b >= p.nb && !zero_past_row) break;
                const uint8_t want = 8 * unit + b < p.nb ? (side ? p.w : p.a)[(size_t)(first + r) * p.nb + 8 * unit + b] : 0;
                wrong += at(side, r)[b] != want;
                ++checked;
            }
    }
}

template <int BM, int BN, int CHUNK>
static void chunks(const Problem& p, bool eager) {
    constexpr int NT = 256;
    using C = ScaleChunks<BM, BN, NT, CHUNK>;
    host.reset(2 * C::BYTES, eager);
    std::vector<C> lanes;
    for (uint32_t t = 0; t < NT; ++t) lanes.emplace_back(p.a.data(), p.w.data(), p.M, p.N, p.nb, p.m0, p.n0, t & 63u, t >> 6, 8 * p.u0);
    auto each = [&](int chunk, auto f) {
        host.chunk = chunk;
        for (uint32_t t = 0; t < NT; ++t) host.lane = t & 63u, f(lanes[t]);
    };
    auto issue = [&](int group, int chunk) { each(chunk, [&](C& c) { for (int i = 0; i < C::NG; ++i) c.issue(i, group, chunk, 0); }); };
    auto read = [&](int unit) {
        compare(p, unit, false, [&](int side, int r) -> const uint8_t* {
            if (r >= (side ? BN : BM)) return nullptr;
            return &host.lds[C::base(unit - p.u0) + ((C::row_at((uint32_t)r) + (side ? C::W_ROWS * CHUNK : 0)) ^ C::at(unit - p.u0))];
        });
    };
    each(0, [&](C& c) { c.issue_first(host.lane, 0); });
    const size_t first = host.flying.size();
    issue(0, 1);
    host.land(host.flying.size() - first);
    read(p.u0);
    for (int u = p.u0; u < p.u1; ++u) {
        host.land();
        if (u + 1 < p.u1) read(u + 1);
        if (u + 2 < p.u1) issue((u - p.u0 + 1) % C::Q, (u - p.u0 + 1) / C::Q + 1);
    }
}

template <int BM, int BN, int UNITS>
static void windows(const Problem& p, bool eager) {
    constexpr int NT = 256;
    using C = ScaleChunkWindows<BM, BN, NT, UNITS>;
    host.reset(2 * C::BYTES, eager);
    std::vector<uint8_t> patch(C::PATCH, 0xEE), dense(C::DENSE_BYTES, 0xEE);
    std::vector<C> lanes;
    for (uint32_t t = 0; t < NT; ++t) lanes.emplace_back(p.a.data(), p.w.data(), p.M, p.N, p.nb, p.m0, p.n0, t, t & ~63u, 8 * p.u0);
    auto each = [&](int chunk, auto f) {
        host.chunk = chunk;
        for (uint32_t t = 0; t < NT; ++t) host.lane = t & 63u, f(lanes[t], t);
    };
    auto issue_group = [&](int group, int chunk) { each(chunk, [&](C& c, uint32_t) { c.issue_group(group, chunk, 0); }); };
    const int patch_from = C::patch_from(p.nb);
    auto bring = [&](int unit, int chunk, int part) {
        const bool tail = unit >= patch_from;
        std::vector<uint3> win(NT * C::G);
        each(-2, [&](C& c, uint32_t t) { for (int g = 0; g < C::G; ++g) win[t * C::G + g] = c.gather(g, chunk, part, host.lds.data(), tail, patch.data()); });
        each(-2, [&](C& c, uint32_t t) { for (int g = 0; g < C::G; ++g) c.put(g, win[t * C::G + g], dense.data(), tail, unit); });
        compare(p, unit, tail, [&](int side, int r) -> const uint8_t* {
            return r < (side ? BN : BM) ? &dense[(size_t)(side ? C::DENSE_W : 0) + 8 * r] : nullptr;
        });
    };
    each(0, [&](C& c, uint32_t) { c.issue_chunk(0, 0); });
    if (C::Q == 1) each(1, [&](C& c, uint32_t) { c.issue_chunk(1, 0); });
    const size_t first = host.flying.size();
    if (C::Q > 1) issue_group(0, 1), issue_group(1, 1);
    if (C::needs_patch(p.M, p.N, p.nb, p.m0, p.n0))
        for (uint32_t t = 0; t < NT; ++t) C::fill_patch(p.a.data(), p.w.data(), p.M, p.N, p.nb, t, patch.data());
    host.land(host.flying.size() - first);
    bring(p.u0, 0, 0);
    if (C::Q == 1) issue_group(0, 2);
    int chunk = C::Q == 1 ? 1 : 0, part = C::Q == 1 ? 0 : 1;
    for (int u = p.u0; u + 1 < p.u1; ++u) {
        bring(u + 1, chunk, part);
        host.land();
        if (++part == C::Q) part = 0, ++chunk;
        if (u + 2 < p.u1) issue_group(part, chunk + 1);
    }
}

// codes of every unit, `column` bytes into the row as with whole rows, or in the lanes' offsets as with rows of any length
template <int BM>
static void codes(int rows, int more, int nb, bool whole) {
    constexpr int NT = 256, ROWS = NT / 8;
    const int M = BM + rows + more;
    const uint32_t pitch = 16u * (uint32_t)nb;
    const std::vector<uint8_t> a = operand(M, (int)pitch, 5u + (uint32_t)nb);
    const CodeRows<ROWS> c(a.data(), M, BM, pitch);
    for (int unit = 0; 8 * unit < nb; ++unit) {
        host.reset(BM * 128, true);
        for (uint32_t t = 0; t < NT; ++t)
            for (int d = 0; d < BM / ROWS; ++d) {
                const uint32_t last = (uint32_t)nb - 1u - 8u * (uint32_t)unit, piece = last < 7 ? min(t & 7u, whole ? 3u : last) : t & 7u;
                host.lane = t & 63u;
                c.issue(d, t / 8 * pitch + 16u * piece + (whole ? 0u : 128u * (uint32_t)unit), whole ? 128u * (uint32_t)unit : 0u,
                        16u * ((uint32_t)(d * NT) + (t & ~63u)));
            }
        for (int r = 0; r < BM && BM + r < M; ++r)
            for (int b = 0; b < 128 && 128 * unit + b < (int)pitch; ++b) {
                wrong += host.lds[(size_t)(128 * r + b)] != a[(size_t)(BM + r) * pitch + 128 * unit + b];
                ++checked;
            }
    }
}

template <int BM, int BN>
static void tile(bool eager) {
    // rows of the tile, and tiles before it; the last tile of an operand whose rows end within it, and a whole one before others
    struct Rows { int a, w, more; } rows[] = {{BM, BN, 0}, {BM, BN, 7}, {1, 1, 0}, {44, 5, 0}, {2, BN - 3, 0}, {BM - 5, 33, 0}};
    for (const auto& s : rows)
        for (int nb : {4, 8, 12, 16, 17, 18, 20, 23, 25, 28, 31, 32, 33, 36, 47, 49, 51, 64, 68, 71, 73, 76}) {
            Problem p = {BM + s.a + s.more, BN + s.w + s.more, nb, BM, BN, 0, 0, {}, {}};
            p.a = operand(p.M, nb, 1u + (uint32_t)nb);
            p.w = operand(p.N, nb, 77u + (uint32_t)nb);
            if (nb % 4 == 0) codes<BM>(s.a, s.more, nb, true), codes<BN>(s.w, s.more, nb, true);
            codes<BM>(s.a, s.more, nb, false), codes<BN>(s.w, s.more, nb, false);
            const int units = (nb + 7) / 8;
            for (int u0 = 0; u0 < units; u0 += 3)
                for (int u1 : {units, u0 + 1}) {
                    p.u0 = u0;
                    p.u1 = u1;
                    if (nb % 4 == 0) chunks<BM, BN, 16>(p, eager), chunks<BM, BN, 32>(p, eager);
                    if (nb >= ScaleChunkWindows<BM, BN, 256, 3>::MIN_NB) windows<BM, BN, 1>(p, eager), windows<BM, BN, 3>(p, eager);
                }
        }
}

int main() {
    for (bool eager : {false, true}) {
        tile<128, 128>(eager);
        tile<192, 128>(eager);
        tile<128, 256>(eager);
        tile<192, 256>(eager);
        tile<256, 256>(eager);
    }
    printf("checked %ld wrong %ld differ %ld past %ld\n", checked, wrong, host.differ, host.past);
    return 0;
}
