// The copies of csrc/lds_dma.h on the host, a lane at a time: they are recorded, checked and land when they are told to.
#pragma once
#include <hip/hip_runtime.h>

#include <stdio.h>
#include <string.h>
#include <vector>

namespace arcq {

struct buffer_t {
    const uint8_t* base;
    uint32_t bytes;
    uint32_t operator[](int i) const { return i == 2 ? bytes : 0; }
};
inline buffer_t buffer_of(const uint8_t* base, uint32_t bytes) { return {base, bytes}; }

struct Host {
    struct Write { uint32_t place; const uint8_t* from; int chunk; };      // a word; from null: zeros
    std::vector<uint8_t> lds;
    std::vector<const uint8_t*> source;     // of every word of LDS, and the chunk that its copy belonged to
    std::vector<int> of_chunk;
    std::vector<Write> flying;
    uint32_t lane = 0;
    int chunk = 0;                          // that copies belong to
    bool eager = false;                     // copies land as soon as they are issued, else in land()
    long differ = 0, past = 0;              // words that copies of one chunk wrote from different places; lanes of copies with a scalar offset past the operand

    void reset(uint32_t bytes, bool eager_) {
        lds.assign(bytes, 0xA5);
        source.assign(bytes / 4, nullptr);
        of_chunk.assign(bytes / 4, -1);
        flying.clear();
        eager = eager_;
    }
    void write(const Write& w) {
        if (w.from) memcpy(&lds.at(w.place + 3) - 3, w.from, 4);
        else memset(&lds.at(w.place + 3) - 3, 0, 4);
    }
    void land(size_t but = 0) {             // all but the youngest words
        const size_t n = flying.size() - but;
        for (size_t i = 0; i < n; ++i) write(flying[i]);
        flying.erase(flying.begin(), flying.begin() + (long)n);
    }
    void copy(const buffer_t& b, uint32_t words, uint32_t voffset, uint32_t soffset, uint32_t lds_wave_base) {
        // a word is in range where its lane's offset is below bytes - scalar offset, which is a number only up to the operand's end
        past += soffset > b.bytes;
        for (uint32_t i = 0; i < words; ++i) {
            const bool in = soffset <= b.bytes && (uint64_t)voffset + 4 * i < b.bytes - soffset;
            const Write w = {lds_wave_base + 4 * words * lane + 4 * i, in ? b.base + soffset + voffset + 4 * i : nullptr, chunk};
            const uint32_t at = w.place / 4;
            if (of_chunk.at(at) == chunk && source[at] != w.from) ++differ;
            of_chunk[at] = chunk;
            source[at] = w.from;
            if (eager) write(w);
            else flying.push_back(w);
        }
    }
};
extern Host host;

inline void copy16(const buffer_t& b, uint32_t voffset, uint32_t soffset0, uint32_t soffset1, uint32_t lds_wave_base) {
    host.copy(b, 4, voffset, soffset0 + soffset1, lds_wave_base);
}
inline void copy16(const buffer_t& b, uint32_t voffset, uint32_t soffset, uint32_t lds_wave_base) { host.copy(b, 4, voffset, soffset, lds_wave_base); }
inline void copy4(const buffer_t& b, uint32_t voffset, uint32_t soffset, uint32_t lds_wave_base) { host.copy(b, 1, voffset, soffset, lds_wave_base); }

}  // namespace arcq
