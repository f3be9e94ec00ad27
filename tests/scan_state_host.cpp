// The scan state's arithmetic, compiled for the host from the library's own source, for test_scan_state_host.py.
#include "../paper_1705_01626_amd/csrc/zvc.hip"

#include <cstdlib>

namespace {
// ScanState's fields as a call of `tiles` tiles finds them (its own constructor reads them on the device).
struct Call {
    alignas(ScanState) unsigned char bytes[sizeof(ScanState)];
    ScanState* st = reinterpret_cast<ScanState*>(bytes);
    Call(WsHeader* hdr, unsigned tiles) {
        st->hdr = hdr;
        st->calls = ScanCalls(hdr->scan_word);
        st->wide = st->calls.wide(tiles) ? 1u : 0u;
        const unsigned long long mark = wide_mark(hdr->wide_calls);
        st->mark0 = st->wide ? static_cast<unsigned>(mark) : narrow_mark(st->calls.call);
        st->mark1 = st->wide ? static_cast<unsigned>(mark >> 32) : st->mark0;
        st->block_shift = block_shift_of(tiles);
    }
    void end(unsigned tiles) {
        st->hdr->scan_word = st->calls.next(tiles, tiles >> st->block_shift).word();
        if (st->wide) ++st->hdr->wide_calls;
    }
};
}  // namespace

extern "C" {
int host_block_shift(unsigned tiles) { return block_shift_of(tiles); }
size_t host_header_bytes() { return kHeaderBytes; }
// The most bytes of scan state that a call for n elements may use: 16 KB tiles, a wide call.
size_t host_scan_bytes(size_t n, int w) { return scan_state_bytes(tiles_for(n, w, kMinLoads)); }

// What a call of `tiles` tiles does to the prefixes in `header`: the prefix of every tile that ends a block, the
// last tile's zeroing.  -1 if the zeroing touches one that the call published; else their number.
int host_prefix_call(unsigned char* header, unsigned tiles) {
    Call call(reinterpret_cast<WsHeader*>(header), tiles);
    const ScanState& st = *call.st;
    unsigned published = 0;
    for (unsigned tile = (1u << st.block_shift) - 1u; tile < tiles; tile += 1u << st.block_shift) {
        if (!st.ends_block(tile)) return -1;
        *st.prefix(tile >> st.block_shift) = st.tag() << kTagShift | tile;
        ++published;
    }
    for (int lane = 0; lane < kWaveSize; ++lane) st.zero_prefixes_left(tiles, lane);
    for (unsigned b = 0; b < published; ++b)
        if (*st.prefix(b) >> kTagShift != st.tag()) return -1;
    call.end(tiles);
    return static_cast<int>(published);
}

// Calls of tiles[0], tiles[1], ... on a workspace with room for `slots` tiles, all of whose counts are written.  Returns the
// first call that would have taken a word from before for one of its counts, or -1.
int host_calls(const unsigned* tiles, int calls, unsigned slots, int* wide_calls) {
    unsigned char* const ws = static_cast<unsigned char*>(std::calloc(1, kHeaderBytes + scan_state_bytes(slots)));
    int bad = -1;
    for (int k = 0; k < calls && bad < 0; ++k) {
        Call call(reinterpret_cast<WsHeader*>(ws), tiles[k]);
        const ScanState& st = *call.st;
        unsigned* const words = st.counts();
        for (unsigned t = 0; t < tiles[k]; ++t)
            if (st.wide ? st.is_there0(words[2 * t]) && st.is_there1(words[2 * t + 1])
                        : t % 2 == 0 ? st.is_there0(words[t]) : st.is_there1(words[t])) bad = k;
        for (unsigned t = 0; t < tiles[k]; ++t) {
            if (st.wide) st.wide_counts()[t] = st.mark() | kCountOwner | t;
            else words[t] = st.mark0 | kCountOwner | t;
        }
        call.end(tiles[k]);
    }
    *wide_calls = static_cast<int>(reinterpret_cast<WsHeader*>(ws)->wide_calls);
    std::free(ws);
    return bad;
}

// Whether a count of 32 bits or 64, or what the pre-pass leaves, passes for the other kinds: bit 0 as a narrow
// one with even or odd index of any call, bit 1 as a wide one of any number.
int host_passes_as(unsigned long long word) {
    const unsigned low = static_cast<unsigned>(word), high = static_cast<unsigned>(word >> 32);
    return (low >> 31 | high >> 31) | (high >> 30 == 1u && low >> 31 == 0u ? 2 : 0);
}
unsigned host_narrow_count(unsigned call, unsigned kept, int owner) { return narrow_mark(call) | (owner ? kCountOwner : 0u) | kept; }
unsigned long long host_wide_count(unsigned long long number, unsigned kept, int owner) {
    return wide_mark(number) | (owner ? kCountOwner : 0u) | kept;
}
unsigned long long host_in_halves(unsigned long long v) { return in_halves(v); }
unsigned long long host_from_halves(unsigned long long v) { return from_halves(v); }
}
