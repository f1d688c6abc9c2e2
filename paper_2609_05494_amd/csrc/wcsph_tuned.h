// Scan shapes of the pair pass, written by paper_2609_05494_amd/autotune.py.
// Workload C2, 1000 timed steps; ms per step of every shape:
//   u128_l24_r1: 0.0795
//   u128_l16_r1: 0.0799
//   u128_l24_r2: 0.0802
//   u128_l16_r2: 0.0806
//   u128_l32_r1: 0.0866
//   u128_l32_r2: 0.0873
// A shape given on the command line (-DUCAP=... when the tuner builds its
// variants) takes precedence over the one recorded here.
#pragma once
#ifndef UCAP
#define UCAP 128
#endif
#ifndef LCAP
#define LCAP 24
#endif
#ifndef RU
#define RU 1
#endif
