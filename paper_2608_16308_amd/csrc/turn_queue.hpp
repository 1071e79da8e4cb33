// An LDS queue that the waves of a workgroup fill over several turns, at most
// TURN entries a turn, and that the whole workgroup empties together.
//
// Emptying takes barriers, so every wave has to come to the same decision at
// the same turn.  A count read while another wave may already add the next
// turn's entries does not give that; here the count is read between two
// barriers, and only at turns for which the room that is known to be left
// (the same number in every thread) no longer suffices.  Between them no wave
// waits for another.
#pragma once
#include <cstdint>

#include "db_format.hpp"

namespace dbs {

// Called by every thread before a turn.  room: places known to be free (CAP
// before the first turn).  True: the caller empties the n entries, sets the
// count to zero and passes a barrier before the turn.
template <uint32_t CAP, uint32_t TURN, class Ops>
DBS_HD bool queue_is_full(uint32_t &room, uint32_t &n, Ops &ops)
{
    static_assert(TURN <= CAP, "a turn fits an empty queue");
    if (room < TURN) {
        ops.barrier();  // the entries of all turns before are in
        n = ops.count();
        ops.barrier();  // and no wave adds until every wave has the count
        if (n > CAP - TURN) {
            room = CAP - TURN;
            return true;
        }
        room = CAP - n;
    }
    room -= TURN;
    return false;
}

}  // namespace dbs
