// Which form of the bf16 attention core a call takes, from the head width, the tokens of a sequence and the (sequence, head) pairs.
// Plain C++: the tests compile it for the host.
#pragma once
#include <cstdint>

namespace sdp {

// workgroups of a launch with one wave along the walked axis (KW = 1: 128 rows each), and of one with several (32 rows)
constexpr int64_t core_blocks_128(int64_t S, int64_t pairs) { return (S + 127) / 128 * pairs; }
constexpr int64_t core_blocks_32(int64_t S, int64_t pairs) { return (S + 31) / 32 * pairs; }

// KW = 4 up to this many workgroups of the KW = 1 form, i.e. while those leave CUs idle: its shorter chains then weigh
// more than the re-reads.  Block forward + backward in us, KW = 1 / KW = 4: heads of 64, 96 workgroups (1 x 1024 tokens,
// 12 heads) 158 / 124, 192 (2 x 1024) 168 / 149, 384 (4 x 1024) 184 / 187; heads of 128, 64 workgroups (1 x 1024, 8 heads)
// 238 / 165, 128 (2 x 1024) 249 / 203, 256 (4 x 1024) 267 / 281; heads of 96, 192 workgroups 208 / 195.
constexpr int64_t core_split_below(int hd) { return hd <= 64 ? 256 : 192; }

// KW = 8 (heads wider than 64): a chain half as long again, two waves on a SIMD where KW = 4 with a workgroup per CU has one, for
// partial results of eight waves to add.  What it shortens grows with S, what it adds with the workgroups: taken from 512 tokens and
// for up to 8 pairs, while KW = 1 has at most 336 workgroups, a round and a third on the chip.  Attention forward + backward of one
// sequence, KW = 1 / 4 / 8 in us, heads of 96: 512 tokens, 4 heads 90 / 52 / 50; 1024, 4 137 / 72 / 65; 1500, 4 180 / 91 / 79; 2048, 4
// 237 / 131 / 109; 2048, 8 247 / 171 / 159; 4096, 2 410 / 200 / 153; 4096, 8 (256 workgroups) 435 / 403 / 348; 6000, 7 (329) 629 / 666 /
// 576; 8192, 2 768 / 440 / 346; 8192, 4 (256) 793 / 689 / 568.  Of 128: 512, 4 104 / 57 / 54; 1024, 4 162 / 80 / 72; 1500, 4
// 214 / 100 / 87; 2048, 4 278 / 149 / 119; 2047, 8 294 / 202 / 185; 4096, 2 486 / 231 / 168; 4096, 4 502 / 307 / 258; 4096, 8 (256)
// 541 / 497 / 428; 6000, 7 (329) 779 / 833 / 744; 8192, 4 (256) 982 / 858 / 700.  Beyond that line KW = 1: 8192, 7 (448) of 96
// 902 / 1188 / 1001, of 128 1080 / 1431 / 1298; 8192, 8 (512) 925 / 1328 / 1087 and 1194 / 1681 / 1371.  Twelve heads of 512 and 1024
// tokens gain nothing (of 96 70.2 / 70.5 and 103.3 / 102.5, KW = 4 / 8), nor do heads of 64 (1 x 512, 8 heads 61 / 62; 1 x 2048 109 /
// 124): their tiles are half as long.
constexpr bool core_in_eight(int hd, int64_t S, int64_t pairs) {
    return hd > 64 && S >= 512 && pairs <= 8 && core_blocks_128(S, pairs) <= 336;
}

// waves along the walked axis: 1, 4 or 8
constexpr int core_waves(int hd, int64_t S, int64_t pairs) {
    return core_in_eight(hd, S, pairs) ? 8 : core_blocks_128(S, pairs) <= core_split_below(hd) ? 4 : 1;
}

// dQ, dK and dV in one launch, where the walked axis is split: saves the gap between two launches and fills the CUs that one of them
// leaves idle, for reading O's rows again (attn_bwd_kernel).  Heads up to 64: up to 384 blocks of 32 rows, and beyond while blocks x tokens,
// which the re-reads grow with, stay within 2^20.  Attention forward and backward, two launches / one, us: 1024 tokens, 8 heads (256
// blocks) 59.7 / 55.9; 1024, 24 (768) 89.1 / 85.2; 2 x 1024, 14 (896) 103.0 / 101.9; 2048, 4 (256) 81.5 / 75.8; 2048, 8 (512) 89.7 / 88.1;
// 4096, 3 (384) 115.4 / 106.9; 8192, 1 (256) 173.9 / 161.5; no difference beyond what runs differ: 2 x 1024, 16 (1024) 107.9 / 108.5, 4096, 4
// (512) 121.2 / 119.0 and 117.9 / 122.0, 8192, 2 (512) 185.0 / 184.3; but 2048, 14 (896) 125.4 / 127.9, 3000, 7 (658) 116.1 / 121.7,
// 4096, 5 (640) 133.8 / 143.1, 6000, 5 (940) 214.8 / 231.5, 8192, 4 (1024) 278.8 / 293.0.
// Wider heads, one workgroup a CU: up to as many blocks as the first half of them fills the CUs.  Of 128: 1024, 8 (256, KW = 8) 91.7 /
// 86.0; 4096, 2 (256) 171.0 / 159.7; but 3000, 3 (282) 149.5 / 152.2; 512, 14 (224, KW = 4) 84.4 / 82.3, but 512, 20 (320) 100.5 / 104.3.
constexpr bool core_merged_backward(int hd, int64_t S, int64_t pairs) {
    const int kw = core_waves(hd, S, pairs);
    const int64_t blocks = core_blocks_32(S, pairs);
    if (kw == 1) return false;
    return hd <= 64 ? blocks <= 384 || blocks * S <= (1 << 20) : blocks <= (kw == 8 ? 256 : 224);
}

} // namespace sdp
