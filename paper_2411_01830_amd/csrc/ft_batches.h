// How the wavefronts of one workgroup share out tickets that the launch's counter hands out in batches: the protocol alone,
// over a memory that the caller supplies, so that it can be run by threads without a GPU.
//
// The workgroup holds one batch in use and at most one drawn ahead. A wavefront takes single tickets out of the batch in
// use; the one that finds it just used up takes the batch ahead into use and from then on owes the draw of the next.
// So tickets are begun in the order of the counter whatever the tiles cost: a wavefront that is late delays its own tile
// and nothing else.
#pragma once
#include <stdint.h>

#include "ft_tables.h"

namespace ft {

constexpr uint32_t kNoBatch = ~0u;

// M: add_taken() adds 1 to the batch word - first ticket << 6 | tickets taken (more than the batch has: it is used up) -
// and returns what it was; word() / set_word(v) read and write it; ahead() / set_ahead(t) do so with the first ticket of
// the batch drawn ahead, kNoBatch if there is none; pause() lets the other wavefronts run. The caller starts with a word of
// `batch` (used up) and a first batch ahead.
//
// Returns the wavefront's next ticket, at or beyond `end` if none is left; *draw: this wavefront owes the next draw, to be
// made and put into ahead() before it calls this again, if its ticket is before `end`.
// Every wait ends: whoever took the batch in use into use owes the draw and makes it without waiting for anybody, unless the
// batch lies at or beyond the end; then it stays where it is, for every wavefront that is still to come.
template <class M>
FT_HD uint32_t take_ticket(M &m, uint32_t batch, uint32_t end, bool *draw) {
  *draw = false;
  for (;;) {
    const uint64_t was = m.add_taken();
    const uint32_t taken = (uint32_t)was & 63;  // at most the batch and one per wavefront
    if (taken < batch) return (uint32_t)(was >> 6) + taken;
    if (taken == batch) {  // exactly one wavefront
      uint32_t first = m.ahead();
      while (first == kNoBatch) {
        m.pause();
        first = m.ahead();
      }
      if (first < end) {
        m.set_ahead(kNoBatch);
        *draw = true;
      }
      m.set_word((uint64_t)first << 6 | 1);
      return first;
    }
    // until there is a next batch: by then its tickets may be taken as well, and this is the wavefront to see to the one after
    while (((uint32_t)m.word() & 63) > batch) m.pause();
  }
}

// Tickets per batch of a workgroup of so many wavefronts. The counter answers 70 million draws a second, and compute units
// that find their source in the last-level cache begin 400 million tiles: with batches of 4 the counter was the limit (419 MB in rows
// of 256 bytes 169 us, 105 MB in rows of 2000 bytes 44 us; batches of 8: 147 and 32 us; of 16: 151 and 35 us).
FT_HD uint32_t wave_batch(uint32_t waves) { return waves < 8 ? waves : 8; }

// Whether a launch of `round` wavefronts shares its tickets out that way. Up to one and a half rounds - most tickets are begun
// at once - a wavefront takes every round-th ticket: the first look at LDS and at the counter would cost what it
// could save (36 MB in rows of 5760 bytes, 4350 tickets for 4096 wavefronts: 12.7 us, shared out 13.8).
FT_HD bool wave_shares(uint64_t round, uint64_t ntickets) { return ntickets > round + round / 2; }

// And whether it then consults the counter at all: workgroup b has batch b behind the first round from the start (63 MB in
// rows of 256 bytes, 7680 tickets for 4096 wavefronts: 19.0 us, with the counter asked all the same 21.3).
FT_HD bool wave_counts(uint64_t workgroups, uint32_t waves, uint64_t ntickets) {
  return wave_shares(workgroups * waves, ntickets) && ntickets > workgroups * (waves + wave_batch(waves));
}

// The last of the launch's draws (they count from 0). A workgroup draws once for every batch that it takes into use before the
// end - one from the start and those that the counter handed it - and so exactly once beyond the end: all draws together
// are the counter's batches and one per workgroup, and who makes the last one may set the counter back.
FT_HD uint32_t wave_last_draw(uint32_t workgroups, uint32_t waves, uint32_t ntickets) {
  const uint32_t batch = wave_batch(waves), left = ntickets - workgroups * (waves + batch);
  return (left + batch - 1) / batch + workgroups - 1;
}

}  // namespace ft
