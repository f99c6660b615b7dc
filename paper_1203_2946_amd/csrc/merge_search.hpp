// Addresses of the sorted conversion's merge search (merge_runs_regs), apart from
// the kernels so that host code can walk them too: constexpr functions of plain
// integers, no HIP in this file.
//
// A group of lanes keeps its strip's words in LDS by place and a table of the
// places its rows start at.  An entry searches the partner run of its own: `cur`
// is the address of the last word known to be below it, one word before the run
// at first, and a step moves it on by a power of two where that stays in the run
// and the word there is below.  Every lane of a wave takes every step, also one
// whose strip the group does not hold, and reads cur + step before it knows
// whether that lies in the run.  So the table must hold places of the group's own
// words for each of its lanes (row_place); a read then lies at most the first
// step past the run, and the first step is at most the words a group can hold.
#pragma once

namespace cmrs {

// Entry `row` of a group's row table: the place the row starts at, n (the strip's
// entries) past the strip's last row and for the entry behind the last.  A strip
// that the group does not hold (`fits` false: none, or longer than its capacity)
// has empty rows at place 0: its pointers are no places of the group's LDS.
constexpr int row_place(bool fits, int row, int nr, int start, int n) {
    return !fits ? 0 : (row < nr ? start : n);
}

// First step, in bytes, of a search in runs of at most `longest` 4-byte words.
constexpr int merge_first_step(int longest) { return longest > 0 ? 4 << (31 - __builtin_clz(longest)) : 0; }

// `cur` after a step: `below` says that the word at cur + step is below the entry's.
constexpr int merge_step(int cur, int step, int last, bool below) {
    return static_cast<int>(cur + step <= last) & static_cast<int>(below) ? cur + step : cur;
}

}  // namespace cmrs
