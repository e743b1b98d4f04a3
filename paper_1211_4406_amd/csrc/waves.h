// How many waves share one group's list (pair.hip, quad.hip).
#pragma once

#include <cstdint>

namespace srf {

// A tree of few groups leaves SIMDs idle, or waiting for its longest list, with
// one wave per group; but waves beyond the work there is cost more than they
// give: a list of fewer tiles than waves is staged by several of them (force,
// potential) or leaves them idle, their LDS taken (adjoint, quadrupole).  So,
// with the pairs per lane of a group's average list (targets x entries / 64):
//   8 waves in trees of at most kEightGroups groups of at least kWavePairs
//     pairs per lane,
//   4 in those of at most kFourGroups of as many, and, up to `reach` groups for
//     each entry of the average list, where the average list has about three
//     tiles (kWaveEntries): whole tiles are dealt then, and the longest lists
//     are several tiles,
//   1 otherwise.
// The limits are the nearest to the best of 1, 4 and 8 waves over 130 sets
// (uniform, clustered and lattice, 1000 to 4 x 10^6 particles, groups of at
// most 1 to 64, cutoffs of 1.6 to 6 spacings): 1-3 % from it on average, and 34 %
// at most (a 20 us call).  Kernel calls with 1 / 4 / 8 waves, us:
//   groups  entries  pairs  force FP32      adjoint FP32    potential FP32  force FP64    adjoint FP64
//   20000   39       0.6    40/94/216       72/154/264      35/77/157       48/126/239    108/273/539
//   87      262      94     37/29/29        59/58/58        36/28/27        46/33/34      66/62/65
//   958     246      80     35/32/40        64/64/86        34/32/37        45/48/64      76/98/154
//   493     323      205    91/45/42        169/87/83       88/44/42        130/58/56     199/100/123
//   250     1517     949    297/96/73       626/198/147     297/95/74       451/139/123   754/237/197
//   2061    383      145    58/55/65        90/96/135       54/49/60        94/88/131     120/157/257
//   3040    1627     1096   411/256/256     831/497/497     418/250/248     734/477/622   1206/829/1003
//   5340    480      176    92/100/127      149/186/298     85/89/119       181/198/296   247/353/630
//   6034    730      248    215/158/195     403/328/427     204/138/178     350/295/448   678/628/975
//   35405   227      40     137/285/543     247/574/1069    117/238/515
//   11262   573      407    248/280/339     452/567/921     221/233/307
//   12715   1504     969    870/702/799     1821/1374/1605  831/635/773
//   21404   1300     978    1009/970/1135   1842/1899/2368  903/833/1106
//   24459   1626     1089   1504/1366/1519  3003/2662/3085  1434/1202/1476
//   43303   425      307    519/680/991     1028/1765/3150  425/556/918
//   50570   1367     886    2327/2302/2823  4620/4778/5980  2248/2201/2895
// and the quadrupole pass, whose work is the lists' cells alone, FP32 and FP64:
//   250     1517            120/83/76       152/99/99
//   3040    1627            229/197/215     364/348/351
//   6034    730             262/251/317     413/493/494
//   12715   1504            418/428/547
//   43303   425             136/198/320
// (By the number of groups alone, 8 below 3500 and 4 below 55000, chosen on
// groups of 64 targets with lists of about 1500 entries, lists of few tiles took
// up to 2.7 times as long as with one wave.)
constexpr int64_t kEightGroups = 700, kFourGroups = 3000;
constexpr double kWavePairs = 90.0, kWaveEntries = 700.0;
// groups per entry of the average list, by kernel
constexpr double kForceReach = 26.0, kAdjointReach = 18.0, kQuadrupoleReach = 5.0;

// ng groups with `entries` list entries and `interactions` (targets x entries)
// in all.
constexpr int waves_per_group(int64_t ng, int64_t entries, int64_t interactions, double reach) {
    const double pairs = (double)interactions / (64.0 * (double)ng), mean = (double)entries / (double)ng;
    if (ng <= kEightGroups && pairs >= kWavePairs) return 8;
    if (ng <= kFourGroups && pairs >= kWavePairs) return 4;
    if (mean >= kWaveEntries && (double)ng <= reach * mean) return 4;
    return 1;
}

}  // namespace srf
