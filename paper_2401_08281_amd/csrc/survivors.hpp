// Places in the list that the survivors of all queries share (kernels_mscan.hip): plain C++, checked on the host as well.
#pragma once

#if defined(__HIPCC__)
#define VS_HOST_DEVICE __host__ __device__
#else
#define VS_HOST_DEVICE
#endif

// A query's `mine` survivors would start at `at` of a list with room for `cap`; places are handed out without gaps, in
// any order of the queries.  full: they do not all fit, and nothing of them is written.  At most one such query starts
// inside the list (the next place handed out lies behind it): unwritten is then what it leaves empty at the list's end.
struct SurvivorPlace { bool full; unsigned unwritten; };
VS_HOST_DEVICE inline SurvivorPlace survivor_place(unsigned at, unsigned mine, unsigned cap) {
  const bool full = mine > 0u && at + mine > cap;
  return {full, full && at < cap ? cap - at : 0u};
}

// Entries of the list that hold a survivor, all of them at its start: `count` places were handed out, `unwritten` of
// those inside the list were left empty.
VS_HOST_DEVICE inline unsigned survivors_written(unsigned count, unsigned cap, unsigned unwritten) {
  return (count < cap ? count : cap) - unwritten;
}
