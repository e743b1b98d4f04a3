// Which walk builds the lists of a tree: one wave or one thread per group
// (lists.hip).
#pragma once

#include <cmath>
#include <cstdint>

namespace srf {

// Both walks look at the same cells.  A thread's is a chain of dependent loads,
// with a wave for 64 groups, which all wait for the longest; a wave's takes a
// load per 64 cells but some 3 to 4 ns of the chip for a group of even the
// shortest list.  So the waves walk trees of at most kFewWalkGroups groups;
// larger ones of at most kWaveWalkGroups where a group looks at enough cells;
// and up to kDeepWalkGroups of such trees where they are deeper than a uniform
// set's by kDeepLevels (clusters: the threads' walks differ most) and the
// groups have kDeepTargets or more targets.
// make_lists by threads / by waves, us (visits: the estimate below):
//   groups  visits  set                                     threads  waves
//   60000   105     uniform, single-particle groups         293      225
//   66306   172     lattice, groups of at most 32           611      296
//   66676   119     clumps of 60, nothing between           265      286
//   80418   66      clumps of 200                           277      352
//   81947   113     uniform, groups of at most 16           424      312
//   90000   105     uniform, single-particle groups         313      308
//     the same moved (refitted)                             354      414
//   95479   174     clustered                               1194     633
//   133334  122     clumps of 60                            325      509
//   160866  69      clumps of 200                           354      653
//   168001  85      uniform, groups of at most 8            467      537
//   169344  190     uniform                                 994      768
//   190000  107     uniform, single-particle groups         409      591
//   185791  235     clustered                               1606     1133
//   262898  142     uniform                                 845      996
//   265973  880     lattice                                 1840     1955
//   299593  280     clustered, 6 levels deeper              2211     1889
//   379204  249     clustered, 6 levels deeper              2445     2287
//   445392  260     clustered, 6 levels deeper              2763     2612
//   564644  260     clustered, 6 levels deeper              3086     3342
//   330377  187     clustered, groups of at most 4          1735     1874
//   400000  213     clustered, single-particle groups       1871     2193
//     the same moved                                        10672    14976
constexpr int64_t kFewWalkGroups = 1 << 16, kWaveWalkGroups = 3 << 16, kDeepWalkGroups = 7 << 16;
constexpr int kDeepLevels = 4;
constexpr int64_t kDeepTargets = 20;
constexpr double kWalkVisits = 150.0, kGroupsPerVisit = 730.0;

// Whether a tree may be walked by waves at some cutoff (it then gets the
// records that they read).
constexpr bool may_wave_walk(int64_t n, int64_t ng, int n_leaf, int max_level) {
    if (ng <= kWaveWalkGroups) return true;
    int uniform_level = 0;   // of a uniform set's leaves
    while ((n >> (3 * uniform_level)) > n_leaf) ++uniform_level;
    return ng <= kDeepWalkGroups && max_level >= uniform_level + kDeepLevels && n >= kDeepTargets * ng;
}

// About the cells that a group looks at, from the cells of each level (cells[L],
// L <= max_level): those of a box as large as an average group's, of n / ng
// random points, and r_cut around it, or as far as their parents are opened, if
// the level's cells lay anywhere.
inline double walk_visits(int64_t n, int64_t ng, const int32_t* cells, int max_level, double r_cut, double theta) {
    const double k = (double)n / (double)ng, box = std::cbrt(1.0 / (double)ng) * (k - 1.0) / (k + 1.0);
    double visits = 0.0;
    for (int L = 1; L <= max_level; ++L) {
        const double side = std::ldexp(1.0, -L);
        double reach = r_cut;
        if (theta > 0.0 && 2.0 * side / theta < reach) reach = 2.0 * side / theta;
        const double in = std::cbrt((double)cells[L]) * (box + 2.0 * reach + side);
        const double v = in * in * in;
        visits += v < (double)cells[L] ? v : (double)cells[L];
    }
    return visits;
}

// Whether waves walk a tree that has their records.
inline bool wave_walk(int64_t n, int64_t ng, const int32_t* cells, int max_level, double r_cut, double theta) {
    if (ng <= kFewWalkGroups) return true;
    const double least = (double)ng / kGroupsPerVisit < kWalkVisits ? (double)ng / kGroupsPerVisit : kWalkVisits;
    return walk_visits(n, ng, cells, max_level, r_cut, theta) >= least;
}

}  // namespace srf
