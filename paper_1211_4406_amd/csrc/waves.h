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
//   20000   39       0.6    37/89/198       67/128/213      32/70/140       45/115/212      96/232/480
//   87      262      94     37/29/28        57/54/55        36/28/27        47/33/34        64/61/64
//   958     246      80     35/33/39        62/59/80        34/31/37        43/47/64        74/94/150
//   493     323      205    90/46/42        170/84/82       87/43/41        129/60/57       198/102/125
//   250     1517     949    297/95/73       622/198/146     298/96/74       446/136/123     748/235/197
//   2061    383      145    57/53/62        88/90/122       53/50/58        94/88/131       124/155/249
//   3040    1627     1096   412/254/256     843/490/506     411/245/246     727/502/626     1189/862/1016
//   5340    480      176    94/99/126       142/164/258     82/86/116       179/197/300     237/340/596
//   6034    730      248    215/156/190     404/304/393     201/138/175     365/302/463     674/624/943
//   35405   227      40     133/276/535     223/490/897     112/230/492
//   11262   573      407    249/276/338     455/560/904     219/234/306
//   12715   1504     969    871/716/809     1753/1407/1574  829/642/771
//   21404   1300     978    1018/970/1118   1928/1930/2353  922/832/1102
//   24459   1626     1089   1471/1394/1510  2944/2676/3042  1417/1204/1471
//   43303   425      307    517/652/990     1045/1737/3093  428/541/919
//   50570   1367     886    2322/2317/2808  4744/4769/5902  2243/2199/2887
// and the quadrupole pass, whose work is the lists' cells alone, FP32 and FP64
// (which takes four for eight):
//   250     1517            119/82/77       152/100
//   3040    1627            222/194/212     359/344
//   6034    730             264/237/301     408/460
//   12715   1504            380/406/536
//   43303   425             141/210/350
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
