// Self-test of the wavefront primitives: each is compared, on the device, with a
// serial evaluation of its definition.  Every access is to an LDS array of a fixed
// length or to the SELFTEST_TABLES tables of SELFTEST_PLACES 16-bit elements behind
// `tab` (16-byte aligned), so the test cannot touch memory it does not own.
#pragma once
#include "wave_ops.hpp"
#include "../../include/vms_replay.h"

const u32 SELFTEST_TABLES = 3, SELFTEST_PLACES = 1216;

// Moves of N tables in global memory: n elements (every length around a block of 8, a step of 64 blocks and
// two steps), moved from the first, the last and inner places.
template <int N>
DI u32 selftest_gblk(uint16_t *tab)
{
    const u32 lane = lane_id();
    uint16_t *a[N];
#pragma unroll
    for (int f = 0; f < N; f++) a[f] = tab + (u32)f * SELFTEST_PLACES;
    const u32 lengths[] = { 1, 7, 8, 9, 15, 16, 511, 512, 513, 519, 520, 1016, 1023, 1024, 1025, 1032 };
    u32 bad = 0;
    for (u32 n : lengths) {
        const u32 places[] = { 0, 6, 7, 8, n / 2, n - 1, n };
        for (u32 pos : places) {
            if (pos > n) continue;
#pragma unroll
            for (int f = 0; f < N; f++)
                for (u32 i = lane; i < SELFTEST_PLACES; i += 64) a[f][i] = (uint16_t)(i < n ? (f + 1) * 20000 - 9 * i : 0);
            wave_sync();
            gblk_shift_up(a, pos, n);
#pragma unroll
            for (int f = 0; f < N; f++) st_one(a[f], pos, (uint16_t)(f + 1));
            tbl_fence();
#pragma unroll
            for (int f = 0; f < N; f++)
                for (u32 i = lane; i < SELFTEST_PLACES; i += 64) {
                    const u32 from = i < pos ? i : i - 1;
                    const uint16_t want = (uint16_t)(i == pos ? f + 1 : i <= n ? (f + 1) * 20000 - 9 * from : 0);
                    if (ld_tab(a[f] + i) != want) bad |= 1u << 18;
                }
            wave_sync();
            gblk_shift_down(a, pos, n + 1);
            tbl_fence();
#pragma unroll
            for (int f = 0; f < N; f++)
                for (u32 i = lane; i < SELFTEST_PLACES; i += 64) {
                    const uint16_t want = (uint16_t)(i < n ? (f + 1) * 20000 - 9 * i : 0);
                    if (ld_tab(a[f] + i) != want) bad |= 1u << 19;
                }
            wave_sync();
        }
    }
    return bad;
}

// Moves inside an array of 32-bit keys (2048 places): up to its end, and down inside [pos, end), around blocks of 4
// keys, groups of 64 blocks and two groups.
template <int G>
DI u32 selftest_keys(u32 *a)
{
    const u32 lane = lane_id();
    const u32 lengths[] = { 1, 3, 4, 5, 255, 256, 257, 511, 512, 513, 1030, 1900 };
    u32 bad = 0;
    for (u32 n : lengths) {
        const u32 places[] = { 0, 3, 4, n / 2, n - 1 };
        for (u32 pos : places) {
            if (pos >= n) continue;
            const u32 ends[] = { pos + 1, pos + 2, (pos + n) / 2 + 1, n - 1, n };
            for (u32 i = lane; i < 2048; i += 64) a[i] = i < n ? 4000 - 2 * i : 0;
            wave_sync();
            key_shift_up<G>(a, pos, n);
            for (u32 i = lane; i < 2048; i += 64)
                if (a[i] != (i <= pos ? 4000 - 2 * i : i <= n ? 4000 - 2 * (i - 1) : 0)) bad |= 1u << 20;
            wave_sync();
            for (u32 end : ends) {
                if (end <= pos || end > n) continue;
                for (u32 i = lane; i < 2048; i += 64) a[i] = i < n ? 4000 - 2 * i : 0;
                wave_sync();
                key_shift_down<G>(a, pos, end);
                for (u32 i = lane; i < 2048; i += 64)
                    if (a[i] != (i >= n ? 0 : i < pos || i >= end - 1 ? 4000 - 2 * i : 4000 - 2 * (i + 1))) bad |= 1u << 21;
                wave_sync();
            }
        }
    }
    return bad;
}

__global__ __launch_bounds__(64) void selftest_kernel(u32 *fail, uint16_t *tab)
{
    __shared__ u32 in[64], out[64];
    __shared__ u64 arr[256];
    __shared__ u64 big[832];
    __shared__ __attribute__((aligned(16))) uint16_t nar[2048];
    __shared__ __attribute__((aligned(16))) u32 nar32[2048];
    const u32 lane = lane_id();
    u32 bad = 0;
    for (u32 round = 0; round < 8; round++) {
        u32 v = (lane * 2654435761u + round * 40503u) ^ (lane << (round & 7));
        v = round == 7 ? 5u : (v >> (round * 3));
        in[lane] = v;
        wave_sync();
        // minimum
        u32 m = wave_min_u32(v), ref = 0xFFFFFFFFu;
        for (int i = 0; i < 64; i++) ref = min(ref, in[i]);
        if (m != ref) bad |= 1;
        // inclusive scan
        u32 tot, s = wave_scan_add(v & 0xFFFF, &tot);
        out[lane] = s;
        wave_sync();
        u32 run = 0;
        for (int i = 0; i < 64; i++) {
            run += in[i] & 0xFFFF;
            if (out[i] != run) bad |= 2;
        }
        if (tot != run) bad |= 4;
        // ballot / rank / lane reads
        u64 b = ballot((v & 1) != 0);
        u32 below = 0;
        for (u32 i = 0; i < lane; i++) below += in[i] & 1;
        if (rank_in(b) != below) bad |= 8;
        if (from_lane(v, (round * 9) & 63) != in[(round * 9) & 63]) bad |= 16;
        // the prefix sum wraps around at 32 bits (it is taken over decreases too)
        u32 wtot, ws = wave_scan_add(0u - v * 0x10001u, &wtot), wrun = 0;
        out[lane] = ws;
        wave_sync();
        for (int i = 0; i < 64; i++) {
            wrun += 0u - in[i] * 0x10001u;
            if (out[i] != wrun) bad |= 2;
        }
        if (wtot != wrun) bad |= 4;
        wave_sync();
    }
    // the minimum in every lane in turn, and a single value to add in every lane in turn: whatever way across the
    // rows a reduction takes, some lane's value needs each of its steps.  The others hold all ones, values with
    // and without bit 31, neighbours of the minimum.
    for (u32 l = 0; l < 64; l++) {
        const u32 mixed = lane * 2654435761u + l;
        const u32 others[] = { 0xFFFFFFFFu, mixed | 0x80000000u, mixed | 1u, 0x80000001u };
        const u32 least[] = { 0xFFFFFFFEu, 0x7FFFFFFFu, 0u, 0x80000000u };
        for (u32 k = 0; k < 4; k++)
            if (wave_min_u32(lane == l ? least[k] : others[k]) != least[k]) bad |= 1;
        u32 tot, s = wave_scan_add(lane == l ? 0x80000001u : 0u, &tot);
        if (s != (lane >= l ? 0x80000001u : 0u)) bad |= 2;
        if (tot != 0x80000001u) bad |= 4;
        // writes of one lane leave the others as they are
        u32 a = lane, b = lane + 100, c = lane + 200, d = lane + 300;
        const u32 one = write_lane(a, 7000 + l, l);
        if (one != (lane == l ? 7000 + l : lane)) bad |= 1u << 16;
        write_lane4(a, b, c, d, 1000 + l, 2000 + l, 3000 + l, 4000 + l, l);
        if (a != (lane == l ? 1000 + l : lane) || b != (lane == l ? 2000 + l : lane + 100) ||
            c != (lane == l ? 3000 + l : lane + 200) || d != (lane == l ? 4000 + l : lane + 300))
            bad |= 1u << 16;
        write_lane3(b, c, d, 5000 + l, 6000 + l, 7000 + l, 63 - l);
        if (b != (lane == 63 - l ? 5000 + l : lane == l ? 2000 + l : lane + 100) ||
            c != (lane == 63 - l ? 6000 + l : lane == l ? 3000 + l : lane + 200) ||
            d != (lane == 63 - l ? 7000 + l : lane == l ? 4000 + l : lane + 300))
            bad |= 1u << 17;
        u32 e = lane + 400;
        a = lane;
        b = lane + 100;
        c = lane + 200;
        d = lane + 300;
        write_lane2(a, e, 1000 + l, 2000 + l, l);
        if (a != (lane == l ? 1000 + l : lane) || e != (lane == l ? 2000 + l : lane + 400)) bad |= 1u << 17;
        write_lane5(a, b, c, d, e, 11, 22, 33, 44, 55, l);
        if (lane == l ? a != 11 || b != 22 || c != 33 || d != 44 || e != 55 : a != lane || b != lane + 100 || c != lane + 200 || d != lane + 300 || e != lane + 400)
            bad |= 1u << 17;
        if (other_lane(lane + 7, (lane + l) & 63) != ((lane + l) & 63) + 7) bad |= 1u << 17;
        // lanes below l hand a value to the lane after them, the others name lane 63 in vain
        const u32 got = to_lane(lane < l ? lane + 9 : 0u, lane < l && lane < 62 ? lane + 1 : 63u);
        if (lane < 63 && got != (lane > 0 && lane - 1 < l ? lane + 8 : 0u)) bad |= 1u << 17;
    }
    // sorted-array helpers on a descending array of 150 keys, followed by zero keys as they require
    for (u32 i = lane; i < 256; i += 64) arr[i] = i < 150 ? (u64)(1000 - 3 * i) << 32 : 0;
    wave_sync();
    if (count_gt(arr, 150, (u64)700 << 32) != 100) bad |= 32;     // 1000-3i > 700  <=>  i < 100
    u32 c1, c2;
    count_gt2(arr, 150, ((u64)700 << 32) | 0xFFFFFFFFu, ((u64)700 << 32) - 1, &c1, &c2);
    if (c1 != 100 || c2 != 101) bad |= 32;
    for (u32 n = 1; n <= 150; n += (n < 70 ? 1 : 7)) {
        for (u32 i = lane; i < 256; i += 64) arr[i] = i < n ? (u64)(1000 - 3 * i) << 32 : 0;
        wave_sync();
        for (u32 probe = 540; probe <= 1003; probe += 1) {
            u64 key = ((u64)probe << 32) - 1;
            u32 ref = count_gt(arr, n, key), r = rank_desc(arr, n, key), r1, r2;
            rank_desc2(arr, n, key + ((u64)2 << 32), key, &r1, &r2);
            if (r != ref || r2 != ref || r1 != count_gt(arr, n, key + ((u64)2 << 32))) bad |= 256;
        }
        // the same ranks with the first search level cached in registers
        Probe pr;
        probe_refresh(pr, arr, n);
        for (u32 probe = 540; probe <= 1003; probe += 1) {
            u64 key = ((u64)probe << 32) - 1;
            if (rank_probe(pr, arr, n, key) != count_gt(arr, n, key)) bad |= 512;
        }
    }
    for (u32 i = lane; i < 256; i += 64) arr[i] = i < 150 ? (u64)(1000 - 3 * i) << 32 : 0;
    wave_sync();
    shift_up(arr, 70, 150);
    st_one(arr, 70u, (u64)12345);
    wave_sync();
    for (u32 i = 0; i < 151; i++) {
        u64 want = i < 70 ? (u64)(1000 - 3 * i) << 32 : (i == 70 ? (u64)12345 : (u64)(1000 - 3 * (i - 1)) << 32);
        if (arr[i] != want) bad |= 64;
    }
    shift_down(arr, 70, 151);
    for (u32 i = 0; i < 150; i++)
        if (arr[i] != (u64)(1000 - 3 * i) << 32) bad |= 128;
    for (u32 i = 151; i < 256; i++)
        if (arr[i] != 0) bad |= 128;                // the spare places stay zero (arr[150] keeps the moved key's copy)
    // the same over many tiles: 700 keys, 64 spare places, moved from places 0, 37 and 699
    for (u32 pos = 0; pos < 700; pos = pos == 0 ? 37 : (pos == 37 ? 699 : 700)) {
        for (u32 i = lane; i < 832; i += 64) big[i] = i < 700 ? (u64)(5000 - 3 * i) << 32 : 0;
        wave_sync();
        shift_up(big, pos, 700);
        st_one(big, pos, (u64)12345);
        wave_sync();
        for (u32 i = 0; i < 701; i++) {
            u64 want = i < pos ? (u64)(5000 - 3 * i) << 32 : (i == pos ? (u64)12345 : (u64)(5000 - 3 * (i - 1)) << 32);
            if (big[i] != want) bad |= 1024;
        }
        for (u32 i = 701; i < 832; i++)
            if (big[i] != 0) bad |= 1024;
        shift_down(big, pos, 701);
        for (u32 i = 0; i < 700; i++)
            if (big[i] != (u64)(5000 - 3 * i) << 32) bad |= 2048;
        for (u32 i = 701; i < 832; i++)
            if (big[i] != 0) bad |= 2048;
    }
    // arrays of narrow keys: block moves and the rank search with 128 probes in registers
    for (u32 n = 5; n <= 1900; n = n < 40 ? n + 1 : n * 3 + 7) {
        for (u32 pos = 0; pos < n; pos = pos < 18 ? pos + 1 : pos * 2 + 3) {
            for (u32 i = lane; i < 2048; i += 64) nar[i] = nar32[i] = i < n ? 4000 - 2 * i : 0;
            wave_sync();
            blk_shift_up(nar, pos, n);
            blk_shift_up(nar32, pos, n);
            st_one(nar, pos, (uint16_t)7);
            st_one(nar32, pos, 7u);
            wave_sync();
            for (u32 i = lane; i < 2048; i += 64) {
                const u32 want = i < pos ? 4000 - 2 * i : (i == pos ? 7u : (i <= n ? 4000 - 2 * (i - 1) : 0u));
                if (nar[i] != want || nar32[i] != want) bad |= 4096;
            }
            wave_sync();
            blk_shift_down(nar, pos, n + 1);
            blk_shift_down(nar32, pos, n + 1);
            for (u32 i = lane; i < 2048; i += 64) {
                const u32 want = i < n ? 4000 - 2 * i : 0u;
                if (nar[i] != want || nar32[i] != want) bad |= 8192;
            }
            wave_sync();
        }
        Probe2<uint16_t> pr;
        pr.refresh(nar, n);
        Probe2<u32> pr32;
        pr32.refresh(nar32, n);
        for (u32 key = 150; key <= 4003; key += 7) {
            u32 ref = 0;
            for (u32 i = 0; i < n; i++) ref += nar[i] > key ? 1u : 0u;
            if (pr.rank(nar, (uint16_t)key) != ref || pr32.rank(nar32, key) != ref) bad |= 16384;
            const u32 b0 = pr.block((uint16_t)key);
            if (b0 > ref || ref - b0 >= 64) bad |= 32768;
        }
    }
    bad |= selftest_keys<1>(nar32);
    bad |= selftest_keys<2>(nar32);
    bad |= selftest_gblk<2>(tab);
    bad |= selftest_gblk<3>(tab);
    u64 any = ballot(bad != 0);
    if (lane == 0) *fail = any ? (bad | 0x80000000u) : 0;
    if (any && bad) atomicOr(fail, bad);
}
