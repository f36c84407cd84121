// Groups of the persistent sequential kernel: which workgroups carry which samples.  Plain C++ beside the kernel, so that the
// arithmetic can be checked without a device.
#pragma once

#ifdef __HIPCC__
#define SJD_HOST_DEVICE __host__ __device__
#else
#define SJD_HOST_DEVICE
#endif

namespace sjd {

struct SeqGroup {
    int index, groups;     // this group, groups in all
    int members, before;   // workgroups of the group, those of them on lower XCDs than the caller's
    int per;               // samples per group (the last groups may have fewer, or none)
};

// The group of the workgroups on XCD `xcc` when count[] workgroups run on each of the eight XCDs: `xpg` neighbouring XCDs that have
// any form a group.  The host chooses xpg for a device of eight XCDs; with fewer (a partition of the device) it is halved until a group's
// share of the B samples is at most max_rows, which is as far as one XCD per group goes.
SJD_HOST_DEVICE inline SeqGroup seq_group_of(const int (&count)[8], int xcc, int xpg, int B, int max_rows) {
    SeqGroup g{};
    int rank = 0, present = 0;
    for (int x = 0; x < 8; ++x) {
        if (x == xcc) rank = present;
        present += count[x] > 0 ? 1 : 0;
    }
    for (;; xpg /= 2) {
        g.groups = (present + xpg - 1) / xpg;
        g.per = (B + g.groups - 1) / g.groups;
        if (g.per <= max_rows || xpg == 1) break;
    }
    g.index = rank / xpg;
    int seen = 0;
    for (int x = 0; x < 8; ++x) {
        if (count[x] <= 0) continue;
        if (seen / xpg == g.index) {
            g.members += count[x];
            if (x < xcc) g.before += count[x];
        }
        ++seen;
    }
    return g;
}

// XCDs per group of the persistent kernel on n_cus workgroups.  More of them spread a stage's weights over more CUs and read them from memory
// fewer times, but only a group of one XCD exchanges through its L2 (0.4 to 1.2 us less an exchange), and a larger group has more
// rows to pass round.  Microseconds a step with 8 / 4 / 2 / 1 XCDs per group: width 512, 4 layers, 256 tokens: one sample 55.6 / 55.6 / 56.2 / 54.5, 4
// samples 59.4 / 57.6 / 57.2 / 56.1, 16 66.3 / 64.0 / 62.0 / 56.9, 64 - / - / 77.1 / 67.6; 8 layers: one sample 104 / 104 / 108 / 106, 5 118 / 111 / 114 / 108; 64 of 1024 tokens
// - / - / 213 / 194; width 256, 6 layers, 37 samples - / - / 92 / 57; width 768, 8 layers, 200 tokens: one sample 119 / 119 / 140 / 179, 32 samples - / 144 / 167 / 192; width
// 1024, 8 layers, 19 samples - / 177 / 206 / 270; 2 layers, one sample 37 / 40 / 45 / 63: from width 768 on one XCD takes longer to pull all
// weights through its L2 than the exchanges of several cost.  So it does at width 512 where a CU mask leaves an XCD fewer CUs; 4 layers, 256 tokens, 2 / 1 XCDs
// per group: 224 CUs, 5, 16, 64 samples 63.1 / 66.2, 65.7 / 66.5, 88.2 / 86.0; 192: 62.3 / 66.2, 63.7 / 66.5, 82.9 / 85.4; 128: 59.0 / 72.1, 59.4 / 73.6, 82.4 / 93.7; 64 CUs, 64
// samples 120 / 156; width 256 on 128 CUs 75 / 60.  A group holds at most sixteen samples (one row block of the matrix
// instruction) unless the batch leaves no choice.
inline int seq_xcds_per_group(int W, int batch, int n_cus = 256) {
    int x = W <= 256 || (W <= 512 && n_cus >= 256) ? 1 : W <= 512 ? 2 : 4;
    if (batch <= 4 && W > 256) x = W <= 512 ? 4 : 8;
    while (x > 1 && (batch * x + 7) / 8 > 16) x /= 2;
    return x;
}

// Whether the first cached rows of a member's first two pairs are requested into LDS between the stages before the attention
// (decode_persistent.hip): one row block per group (two leave no room), widths from 512 on (narrower ones have no such kernel), the busiest members
// with a second pair, and a prefix long beside the weights that those stages load.  The requests cost every member, and a member with one
// pair waits for one set of cached rows at most.  The line of width 512 was drawn for groups of two XCDs; those of one have shorter exchanges and less idle
// time, and for them it lies too low below 1024 tokens, by 8 % of a step at 256.  Microseconds a step without -> with, busiest group's pairs / members:
//   width 512, 4 layers, one XCD per group: 256 tokens: 24/32 57.4 -> 63.0, 48/32 60.6 -> 65.2, 64/32 62.5 -> 67.5, 96/32 73.4 -> 78.7, 128/32 80.0 -> 84.7; 600: 64/32
//     76.3 -> 78.8, 128/32 113.9 -> 112.9; 1024: 32/32 73.5 -> 78.2, 40/32 85.8 -> 87.6, 48/32 89.5 -> 89.4, 64/32 99.0 -> 98.3, 128/32 151.0 -> 147.8; 2048: 32/32
//     101.4 -> 103.5, 48/32 131.1 -> 128.2; 4096: 24/32 133.8 -> 137.6, 64/32 232.8 -> 229.7; 8 layers: 256 tokens, 64/32 123.9 -> 133.1, 1024 195.8 -> 193.7;
//   two XCDs (where a CU mask leaves fewer CUs; these on all of them): 256 tokens: 64/64 64.0 -> 66.8, 72/64 69.7 -> 71.4, 80/64 72.0 -> 72.8, 88/64 74.5 -> 74.7, 96/64
//     76.1 -> 75.1, 128/64 79.9 -> 77.8, 256/64 99.1 -> 97.3; 1024: 64/64 78.0 -> 81.4, 88/64 99.7 -> 97.4, 128/64 116 -> 109; 192: 128/64 78.1 -> 76.6, 200/64 90.1 -> 90.9;
//   width 768, 8 layers: 513 tokens: 132/128 150.1 -> 152.6, 156/128 162.3 -> 164.9; 600: 144/128 166.5 -> 166.9, 168/128 174.7 -> 174.3, 192/64 229.0 -> 229.1;
//     777: 144/128 177.5 -> 177.2, 168/128 186.0 -> 184.0, 120/128 159.9 -> 162.8; 4 layers, one XCD: 600 tokens, 192/32 171.0 -> 170.8, 1024 219.5 -> 216.9;
//   width 1024, 8 layers: 513 tokens: 128/128 176.2 -> 180.4, 144/128 193.4 -> 190.6, 256/128 221 -> 211; 777: 160/128 222.3 -> 215.2; 4 layers, one XCD: 513 tokens, 256/32
//     242 -> 244, 777 290 -> 290.
inline bool seq_rows_ahead(int B, int heads, int width, int T, int n_cus, int xpg) {
    if (B > 128 || width < 512 || T < (width <= 512 ? 256 : width <= 768 ? 600 : 513)) return false;
    const int groups = 8 / xpg, members = n_cus / groups, pairs = (B + groups - 1) / groups * heads;
    return width <= 512 ? 8 * pairs >= 11 * members : pairs > members;
}

}  // namespace sjd
