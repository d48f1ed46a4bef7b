// Counters of the FP32 pair walk's partner rings.
#pragma once

namespace csph {

// One lane's write and read counters in bytes, SLOT per entry: a slot's address is the counter
// masked to the ring (RING bytes, a power of two), and the write counter gives |N(i)| without a
// count of its own.  The walk tells it of its pops and settles the counters well before 32 bits
// of them are used up.  constexpr: host and device code alike.
template <unsigned SLOT, unsigned RING>
struct RingCount {
    unsigned qw = 0, qr = 0;
    int drop = 0, ghosts = 0;  // entries that do not count: turned down (less those settled), mirror
    unsigned pops = 0;         // pops since the counters were settled, by any lane (wave-uniform)

    // pops a lane may make before its counters are settled; the drains between two looks, a few
    // hundred, and the ring's own entries come on top
    static constexpr unsigned kPops = 1u << 20;
    static_assert((kPops + (1u << 16)) < 0xffffffffu / SLOT, "counters of 32 bits");

    constexpr void popped(unsigned n) { pops += n; }
    // The entries popped leave the counters for `drop`, in whole rings: the slots stay in place.
    constexpr void settle_counters() {
        if (pops < kPops) return;
        pops = 0;
        const unsigned d = qr & ~(RING - 1u);
        qw -= d;
        qr -= d;
        drop -= (int)(d / SLOT);
    }
    // |N(i)|: the entries queued less the mirror entries and those the FP64 test turned down
    constexpr int count() const { return (int)(qw / SLOT) - ghosts - drop; }
};

}  // namespace csph
