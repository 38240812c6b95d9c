// How long a block of the rejection half naps between two polls of a bounded wait, in units of 64 clocks.
#pragma once

// The limit of a wait is a number of polls, so the long nap is what its time comes from: shorter ones are for the
// first polls only.
// short_naps: in a small launch the data is a poll or two away and a long nap would be most of the wait.  In a large one many
// blocks wait at once and their polls compete with the streams (short naps there: the 7B- and 70B-shaped steps 0.5
// to 0.8% slower).
// few: few blocks wait like this (the final stage's, at the very end), so that their polls cost the streams nothing
// (rejection alone, one request 12.7 -> 12.2 us, 32 at k = 4 19.4 -> 18.9; the smallest fp32 step 12.7 -> 12.1).
constexpr int kFewNapPolls = 4096;   // a few milliseconds, longer than any healthy launch leaves the final stage waiting
constexpr int nap_length(int poll, bool few, bool short_naps)
{
    return short_naps && poll < 4 ? 2 : ((few && poll < kFewNapPolls) || (short_naps && poll < 8) ? 8 : 32);
}
