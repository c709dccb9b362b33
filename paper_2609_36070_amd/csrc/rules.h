// Which path a forward takes: rules on sizes alone, host code without HIP.
#pragma once

// Dense routing on few token tiles: the folded down product has one workgroup
// per 256 x 256 tile of Y and a K loop over every expert, so a short batch
// leaves most CUs idle (200 tokens at d 7168: 28 workgroups of 288 K steps).
// The experts' products can run as tiles of their own into fp32 instead, with a
// small kernel that adds them in the same order of experts.  That shortens the
// chain of K steps from E f / 64 to `rounds` f / 64, rounds of the 256 CUs
// that E products of Y's tiles take, and costs a write and a read of fp32
// products, (E + shared) T d of them.  A K step of 64 takes about 1.4 us and
// the fp32 traffic runs at about 4.5 TB/s, so the two meet near 12000 values
// per column of f that the chain is shorter by.  Forward, folded / in parts
// (us): 8 experts and a shared one of 2048, d 7168: 200 tokens 706 / 387, 500
// 737 / 494; 8 of 1024, d 1024: 2048 tokens 253 / 128, 8192 450 / 481; 16 of
// 2048, d 256: 8192 tokens 1194 / 636; 8 of 256, d 1024: 2048 tokens 84 / 68,
// 8192 125 / 203; 2 of 256, d 256: 30000 tokens 49 / 71; over 306 shapes of 2
// to 16 experts the line is at most 10 % off the better side.
// Only up to half of the CUs' worth of Y tiles: past them the folded product
// fills the chip itself.
constexpr long DENSE_PARTS_MAX = 128, DENSE_PARTS_VALUES = 12000;

inline bool dense_parts(long T, long d, long E, long k, long f, long fs) {
    const long nt = (T + 255) / 256 * (d / 256);
    if (k != E || T <= 0 || nt > DENSE_PARTS_MAX) return false;
    const long rounds = (E * nt + 255) / 256;
    return (E + (fs > 0)) * T * d < DENSE_PARTS_VALUES * f * (E - rounds);
}
