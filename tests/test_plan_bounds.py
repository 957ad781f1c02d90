"""Every address the GEMM kernels form under the launch configurations the library picks stays inside the buffers
the caller handed over -- checked on the host, for every kernel family, over a grid of shapes.

A host model walks each launch the way its kernel does: the same partition of the work over workgroups (taken from
the library's own qoq_query_gemm_config and qoq_gemm_workspace_bytes), the same iteration structure and tiles (csrc/qoq_tiles.h,
qoq_walk.h, qoq_workspace.h, the headers the library itself includes), the same clamps for rows past M, groups past the end of a run or slice,
fragments past N, and the copies issued past the end of a run.  Each global address the model forms -- packed codes,
level-2 metadata, channel scales and zeros, INT8 activations, token scales and sums, partial tiles and counters in the
workspace -- is checked against the size of its buffer.  The counters of every plan lie in one area of the workspace and
every plan's partial tiles behind it, so no call finds the sums of a call of another shape where it expects counters.  A copy that read group G of the last token row (128 bytes
past the activations) once went unnoticed until it faulted on the GPU; this test makes that class of mistake fail
on the CPU."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

CHECKER = r'''
#include "qoq_layout.h"
#include "qoq_tiles.h"
#include "qoq_walk.h"
#include "qoq_workspace.h"
#include <algorithm>
#include <cstdio>
#include <cstdlib>
#include <vector>
using namespace qoq;
typedef long long ll;
static ll M, N, K, G, ws_bytes; static const ll counters_bytes = kCounterBytes; static int mode, tile, split;
static ll n_codes, n_meta, n_scales, n_zeros, n_qx, n_sx, n_rs;
static const char* fail = nullptr; static ll fail_off, fail_len, fail_size;
static ll parts_end;                                                   // of the partial tiles that the plan touches
static inline void chk(const char* what, ll off, ll len, ll size) {
    if (what[0] == 'p') parts_end = std::max(parts_end, off + len);
    if (!fail && (off < 0 || off + len > size)) { fail = what; fail_off = off; fail_len = len; fail_size = size; }
}
static ll cdiv(ll a, ll b) { return (a + b - 1) / b; }

// ---- LDS-staged and register-streaming kernels: units = (64-channel block, group) dealt in runs ----------------
static void check_stream(int MF, bool staged) {
    const ll blocks = N / 64, total = blocks * G, nwg = split, upw = stream_units_per_workgroup(M, N, G, 16 * MF, nwg), nf_total = N / 16, m_tiles = cdiv(M, 16 * MF);
    const ll kEl = MF * 256;                                   // int4 elements of a partial tile
    for (ll mt = 0; mt < m_tiles; ++mt) for (ll wg = 0; wg < nwg; ++wg) {
        const ll m0 = mt * 16 * MF;
        const int u0 = (int)std::min(total, wg * upw), u1 = (int)std::min(total, u0 + upw);
        if (u0 >= u1) continue;
        RunShape run = make_run(u0, u1, (int)G, staged ? 2 : 8);
        for (int it = 0; it < run.T; ++it) {                   // copies past the end of the run repeat iteration T-1
            const IterInfo o = run_iteration(run, it);
            if (staged) {
                for (int e = 0; e < 2; ++e) {
                    const ll gsel = std::min<ll>(o.g + (e < o.n ? e : 0), G - 1);
                    for (int f = 0; f < 4; ++f) chk("codes", ((o.block * 4 + f) * G + gsel) << 10, 1024, n_codes);
                    for (int b = 0; b < 2 * MF; ++b) for (int r = 0; r < 16; ++r) {
                        const ll row = std::min(m0 + (b >> 1) * 16 + r, M - 1);
                        chk("qx", row * K + gsel * kGroup + (b & 1) * 64, 64, n_qx);
                    }
                    if (mode == 0) chk("meta", gsel * nf_total * 32 + (ll)o.block * 128, 128, n_meta);
                }
                chk("scales", (ll)o.block * 128, 128, n_scales);
                if (mode == 1) chk("zeros", (ll)o.block * 64, 64, n_zeros);
            } else {
                for (int w = 0; w < o.n; ++w) {
                    const ll g = o.g + w;
                    for (int f = 0; f < 4; ++f) {
                        const ll nf = (ll)o.block * 4 + f;
                        chk("codes", (nf * G + g) * 1024, 1024, n_codes);
                        if (mode == 0) chk("meta", (g * nf_total + nf) * 32, 32, n_meta);
                    }
                    for (int mf = 0; mf < MF; ++mf) for (int r = 0; r < 16; ++r)
                        chk("qx", std::min(m0 + mf * 16 + r, M - 1) * K + g * kGroup, 128, n_qx);
                }
            }
            if (o.seg_end) {                                    // epilogue constants / partial tile of the block
                chk("scales", (ll)o.block * 128, 128, n_scales);
                if (mode == 1) chk("zeros", (ll)o.block * 64, 64, n_zeros);
                if (!o.complete) {
                    chk("counter", (mt * blocks + o.block) * 4, 4, counters_bytes);
                    const ll wf = ((ll)o.block * G) / upw, wl = ((ll)o.block * G + G - 1) / upw;   // contributors
                    for (ll ww = wf; ww <= wl; ++ww) for (int which = 0; which < 2; ++which)
                        chk("parts", counters_bytes + ((mt * nwg + ww) * 2 + which) * kEl * 16, kEl * 16, ws_bytes);
                }
            }
        }
        chk("sx", std::min(m0 + 16 * MF - 1, M - 1) * 2, 2, n_sx);
    }
}

// ---- blocks in lockstep: whole pairs / quads per workgroup ---------------------------------------------------------
static void check_lockstep(int NB, int MF) {
    const ll sets = N / (64 * NB), upw = cdiv(sets, split), nf_total = N / 16, m_tiles = cdiv(M, 16 * MF);
    if (N % (64 * NB)) { fail = "lockstep width"; return; }
    for (ll mt = 0; mt < m_tiles; ++mt) for (ll wg = 0; wg < split; ++wg) {
        const ll m0 = mt * 16 * MF, sb0 = std::min(sets, wg * upw), sb1 = std::min(sets, sb0 + upw);
        if (sb0 >= sb1) continue;
        const ll T = (sb1 - sb0) * ((G + 1) / 2);
        ll csb = sb0, cg = 0, cleft = T;
        for (ll it = 0; it < T + 2; ++it) {                   // the copy front, kRing - 1 issues past the end included
            const int two = cg + 1 < G ? 1 : 0;
            for (int pk = 0; pk < 2; ++pk) {
                const ll gsel = cg + (pk & two);
                for (int b = 0; b < 2 * MF; ++b) for (int r = 0; r < 16; ++r)
                    chk("qx", std::min(m0 + (b >> 1) * 16 + r, M - 1) * K + gsel * kGroup + (b & 1) * 64, 64, n_qx);
                if (mode == 0) chk("meta", gsel * nf_total * 32 + csb * NB * 128, NB * 128, n_meta);
                for (int f = 0; f < 4 * NB; ++f) chk("codes", ((csb * 4 * NB + f) * G + gsel) << 10, 1024, n_codes);
            }
            chk("scales", csb * NB * 128, NB * 128, n_scales);
            if (mode == 1) chk("zeros", csb * NB * 64, NB == 2 ? 128 : 256, n_zeros);
            if (cleft > 1) { --cleft; cg += 2; if (cg >= G) { cg = 0; ++csb; } }
        }
    }
}

// ---- activation-stationary kernels ---------------------------------------------------------------------------------
// Non-temporal weights come by buffer loads through a window of the codes of 2 R fragments of the run and one of all metadata: what a wave needs
// is inside, at the unit's own place, and what it does not (slots past the slice, fragments past the run) past the end of the window.
static void check_windows(ll f0, ll nfr, ll g_lo, ll g_hi, ll waves, ll jeff, ll J, ll R) {
    const ll nowhere = 0x80000000ll, nf_total = N / 16, whole = G * nf_total * 32;
    if (whole >= nowhere) { fail = "metadata window"; return; }
    for (ll fi0 = 0; fi0 < nfr; fi0 += R) {
        const ll window = std::min(nfr - fi0, 2 * R) * G * 1024;
        chk("codes", (f0 + fi0) * G * 1024, window, n_codes);
        for (int w = 0; w < waves; ++w) for (ll j = 0; j < J; ++j) for (ll ahead = fi0 == 0 ? 0 : R; ahead < 2 * R; ++ahead) {
            const ll g = g_lo + w * jeff + j;
            const bool valid = j < jeff && g < g_hi, needed = valid && fi0 + ahead < nfr;
            const ll at = (valid ? g * 1024 : nowhere) + ahead * G * 1024, at_m = (valid ? (g * nf_total + f0) * 32 : nowhere) + (fi0 + ahead) * 32;
            if (needed ? at + 1024 > window || (f0 + fi0) * G * 1024 + at != ((f0 + fi0 + ahead) * G + g) * 1024 : at < window) { fail = "codes window"; return; }
            if (at + 1024 > (ll)1 << 32 || at_m + 32 > (ll)1 << 32) { fail = "window offset"; return; }
            if (mode == 0 && needed) chk("meta", at_m, 32, n_meta);
            if (!valid && at_m < whole) { fail = "metadata window"; return; }
        }
    }
}
// Weights, constants and partial tiles of a workgroup's fragments: `waves` waves of jeff groups each (J as compiled, R fragments ahead), kEl int4
// per tile.
static void check_fragments(ll nwg, ll waves, ll S, ll gps, ll m_tiles, ll kEl, ll J, ll R) {
    const bool pass_by = weights_pass_by(N, K, m_tiles, S == 1 ? kPassByWhole : kPassBy);
    const ll nf_total = N / 16, base = nf_total / nwg, rem = nf_total - base * nwg, jeff = cdiv(gps, waves);
    for (ll mt = 0; mt < m_tiles; ++mt) for (ll sl = 0; sl < S; ++sl) for (ll wg = 0; wg < nwg; ++wg) {
        const ll f0 = wg * base + std::min(wg, rem), f1 = f0 + base + (wg < rem ? 1 : 0), g_lo = sl * gps, g_hi = std::min(G, g_lo + gps);
        if (g_lo >= g_hi) { fail = "astat empty slice"; return; }
        if (S > 1 && f1 - f0 > 128) { fail = "astat fragments"; return; }
        if (pass_by) check_windows(f0, f1 - f0, g_lo, g_hi, waves, jeff, J, R);
        for (ll nf = f0; nf < f1; ++nf) {
            for (int w = 0; w < waves; ++w) for (ll j = 0; j < jeff + 3; ++j) {   // slots past jeff re-read the last group
                const ll g = std::min(g_lo + w * jeff + std::min(j, jeff - 1), g_hi - 1);
                chk("codes", (nf * G + g) * 1024, 1024, n_codes);
                if (mode == 0) chk("meta", (g * nf_total + nf) * 32, 32, n_meta);
            }
            chk("scales", ((nf >> 2) * 64 + 48 + 4 * (nf & 3)) * 2, 8, n_scales);
            if (mode == 1) chk("zeros", (nf >> 2) * 64 + 48 + 4 * (nf & 3), 4, n_zeros);
            if (S > 1) {
                chk("counter", (mt * nf_total + nf) * 4, 4, counters_bytes);
                chk("parts", counters_bytes + ((mt * nf_total + nf) * S + sl) * kEl * 16, kEl * 16, ws_bytes);
            }
        }
    }
}
static void check_astat(int tl) {
    const ll m_tiles = cdiv(M, tl);
    if (tl == 64 && M <= 48 * m_tiles) tl = 48;               // as many tiles of 48 tokens
    const bool deep = tl == 16 && G > 64 && G <= 112;          // sixteen waves of seven groups hold all of K
    const ll MF = tl / 16, waves = deep ? 16 : 8, cap = deep ? 112 : tl >= 48 ? 32 : 64, stage = 128 * 1024 / waves;
    ll S = cdiv(G, cap), gps = cdiv(G, S); S = cdiv(G, gps);
    const ll jeff = cdiv(gps, waves), rows = tl == 16 && M <= 8 ? 8 : 16;
    const ll J = deep ? (gps <= 96 ? 6 : 7) : tl >= 48 ? std::max<ll>(jeff, 2) : jeff <= 4 ? 4 : 8;   // groups per wave, as compiled
    if (jeff > J || J * MF > 16) { fail = "astat capacity"; return; }
    // the activation preload, the same for every workgroup of a token tile and slice
    const ll JP = (J >= 8 && waves == 8) || (J > 4 && rows == 8) ? 8 : 4, RP = rows == 8 ? 8 : std::min<ll>(128 / JP, MF * 16);
    const ll row_passes = rows == 8 ? 1 : cdiv(MF * 16, RP), j_passes = cdiv(J, JP), dma = RP * JP / 8;
    if (dma * 1024 > stage || 2 * waves * MF * 1024 > 128 * 1024) { fail = "astat staging"; return; }
    for (ll mt = 0; mt < m_tiles; ++mt) for (ll sl = 0; sl < S; ++sl) {
        const ll m0 = mt * tl, g_lo = sl * gps, g_hi = std::min(G, g_lo + gps);
        if (m0 >= M) { fail = "astat token tile"; return; }
        for (int w = 0; w < waves; ++w) for (ll rp = 0; rp < row_passes; ++rp) for (ll jp = 0; jp < j_passes; ++jp) {
            std::vector<char> copied(dma * 64);
            for (ll i = 0; i < dma; ++i) {
                if (rows == 16 && rp * RP + i * 8 / JP >= MF * 16) continue;   // 48 tokens: half of the second pass
                for (ll flat = i * 64; flat < i * 64 + 64; ++flat) {
                    const ll row_local = flat / (JP * 8), pos = flat % (JP * 8);
                    const ll row = std::min(m0 + rp * RP + row_local, M - 1);
                    const ll col = std::min((g_lo + w * jeff + jp * JP) * kGroup + ((pos ^ (row_local & 15)) * 16), K - 16);
                    chk("qx", row * K + col, 16, n_qx);
                    copied[flat] = 1;
                }
            }
            for (ll mm = 0; mm < RP / rows; ++mm) for (ll jj = 0; jj < JP; ++jj) for (int lane = 0; lane < 64; ++lane) for (int ks = 0; ks < 2; ++ks) {
                const ll j = jp * JP + jj;
                if (j >= J || rp * (RP / rows) + mm >= MF || j >= jeff || g_lo + w * jeff + j >= g_hi) continue;
                const ll row_local = mm * 16 + (lane & 15 & (rows - 1)), at = row_local * JP * 8 + ((jj * 8 + ks * 4 + (lane >> 4)) ^ (row_local & 15));
                chk("staging", at * 16, 16, dma * 1024);
                if (!fail && !copied[at]) { fail = "staging, not copied"; return; }
            }
        }
    }
    check_fragments(split, waves, S, gps, m_tiles, MF * 64, J, deep || J == 8 ? 1 : 2);
}
// Few short tokens, quantized by every workgroup in front of its first fragment (512 threads).
static void check_linear() {
    ll rows = 1, log = 0;
    while (rows < M) { rows *= 2; ++log; }
    const ll per_row = 512 / rows, chunks = rows * K <= 2 * 8 * 512 ? 2 : 8;   // as compiled
    if (M > 16 || rows * K > 32768 || G > 64) { fail = "linear capacity"; return; }
    std::vector<char> made(M * K / 8);
    for (ll t = 0; t < 512; ++t) for (ll i = 0; i < chunks; ++i) {
        const ll row = t >> (9 - log), c = (t & (per_row - 1)) + i * per_row;
        if (row >= M || c >= K / 8) continue;
        chk("x", (row * (K / 8) + c) * 16, 16, M * K * 2);
        chk("LDS codes", row * K + (((c >> 1) ^ (row & 7)) * 16) + (c & 1) * 8, 8, 32768);
        chk("qx", (row * (K / 8) + c) * 8, 8, n_qx);
        made[row * (K / 8) + c] = 1;
    }
    for (char m : made) if (!m) { fail = "linear, a chunk left out"; return; }
    const ll jeff = cdiv(G, 8);
    for (int w = 0; w < 8; ++w) for (ll j = 0; j < jeff && w * jeff + j < G; ++j) for (int lane = 0; lane < 64; ++lane) for (int ks = 0; ks < 2; ++ks) {
        const ll row = std::min<ll>(lane & 15, M - 1);
        chk("LDS codes", row * K + ((((w * jeff + j) * 8 + ks * 4 + (lane >> 4)) ^ (row & 7)) * 16), 16, M * K);
    }
    check_fragments(std::min<ll>(N / 16, 256), 8, 1, G, 1, 64, jeff <= 4 ? 4 : 8, jeff <= 4 ? 2 : 1);
}

// ---- eight waves on equal token tiles ------------------------------------------------------------------------------
static int swizzle(int row) { return (row >> 1) & 7; }
static void check_mma8() {
    const ll MF = eight_wave_fragments(M), TM = 16 * MF, TN = eight_wave_width(M, N, split), WC = TN / 64, WK = 8 / WC, SG = WK / 2;
    const ll kUnits = TN / 16, ABytes = SG * TM * 128, WBytes = SG * TN * 64, Slab = ABytes + WBytes + 512, EBytes = 2304;
    const ll R = 4 * Slab + EBytes <= 160 * 1024 ? 4 : 3, ring = std::max(R * Slab, 16 * MF * 1024);
    const ll n_tiles = cdiv(N, TN), m_tiles = cdiv(M, TM), tiles = n_tiles * m_tiles, S = split, gps = cdiv(G, S), nf_total = N / 16;
    if (MF < 3 || MF > 9 || ring + EBytes > 160 * 1024 || cdiv(G, gps) != S) { fail = "mma8 shape"; return; }
    // LDS, the same for all tiles: copies into a slab, reads of one, the exchange of the waves' sums
    const ll kACopies = SG * TM / 8, kAMost = cdiv(kACopies, 8);
    for (int wave = 0; wave < 8; ++wave) {
        const ll kw = wave % WK, wc = wave / WK, sg = kw >> 1, half = kw & 1;
        for (ll k = 0; k < kAMost; ++k) {
            const ll i = std::min(k * 8 + wave, kACopies - 1);
            chk("LDS activations", i / (TM / 8) * TM * 128 + i % (TM / 8) * 1024, 1024, ABytes);
        }
        for (int u = 0; u < 2; ++u) chk("LDS weights", ABytes + (wave * 2 + u) * 1024, 1024, ABytes + WBytes);
        for (int lane = 0; lane < 64; ++lane) {
            const int r16 = lane & 15, kb = lane >> 4;
            for (ll tf = 0; tf < MF; ++tf)
                chk("LDS activation operands", sg * TM * 128 + r16 * 128 + ((4 * half + kb) ^ swizzle(r16)) * 16 + tf * 2048, 16, (sg + 1) * TM * 128);
            for (ll f = 0; f < 4; ++f) {
                chk("LDS weight operands", ABytes + (sg * kUnits + wc * 4 + f) * 1024 + lane * 16 + half * 8, 8, ABytes + WBytes);
                chk("LDS metadata", ABytes + WBytes + sg * 256 + wc * 128 + f * 32 + (r16 >> 1) * 4, 4, Slab);
            }
        }
        ll lo = 0, hi = MF;
        for (ll bit = WK / 2; bit >= 1; bit >>= 1) {
            const ll mid = (lo + hi + 1) / 2, upper = 4 * (hi - mid) * 64, pair = (((wave >> 1) & ~(bit - 1)) | (wave & (bit - 1))) * 4 * MF * 64;
            const ll give = wave & bit ? mid - lo : hi - mid, take = wave & bit ? hi - mid : mid - lo;
            chk("LDS exchange", pair * 16, ((wave & bit ? upper : 0) + 4 * give * 64) * 16, ring);
            chk("LDS exchange", pair * 16, ((wave & bit ? 0 : upper) + 4 * take * 64) * 16, ring);
            if (4 * (give + take) > 4 * MF) { fail = "exchange area"; return; }
            if (wave & bit) lo = mid; else hi = mid;
        }
    }
    std::vector<char> seen(tiles);
    for (ll b = 0; b < tiles; ++b) {
        const ll xcd = b & 7, slot = b >> 3, q = tiles >> 3, r = tiles & 7, L = xcd * q + std::min(xcd, r) + slot;
        const ll panel = L / (4 * n_tiles), rows = std::min<ll>(4, m_tiles - panel * 4), rem = L - panel * 4 * n_tiles;
        const ll tni = rem / rows, tmi = panel * 4 + rem % rows, m_base = tmi * TM, n_base = tni * TN, nf_base = tni * kUnits;
        if (tni >= n_tiles || tmi >= m_tiles || seen[tmi * n_tiles + tni]++) { fail = "tile order"; return; }
        for (int d = 0; d < 256; ++d) {                        // epilogue constants: 256 of each, clamped
            if (d < 128) chk("sx", m_base * 2 + std::min<ll>(d, (M - m_base - 1) >> 1) * 4, 4, n_sx);
            if (d < 128) chk("scales", n_base * 2 + std::min<ll>(d, ((N - n_base) >> 1) - 1) * 4, 4, n_scales);
            if (mode == 1) chk("rowsum", (m_base + std::min<ll>(d, M - m_base - 1)) * 4, 4, n_rs);
            if (mode == 1 && d < 64) chk("zeros", n_base + std::min<ll>(d, ((N - n_base) >> 2) - 1) * 4, 4, n_zeros);
        }
        for (ll sl = 0; sl < S; ++sl) {
            const ll g_first = sl * gps, Gs = std::min(G - g_first, gps), g_last = g_first + Gs - 1, T = cdiv(Gs, SG);
            if (Gs < 1) { fail = "mma8 empty slice"; return; }
            for (ll st = 0; st <= T; ++st) {                   // activations of stages 0 .. T-1, weights of 0 .. T (bundle T-1 holds those of T)
                for (ll sg = 0; sg < SG; ++sg) {
                    const ll g = std::min(g_first + st * SG + sg, g_last);
                    if (st < T) for (ll rb = 0; rb < TM / 8; ++rb) for (int r8 = 0; r8 < 8; ++r8)
                        chk("qx", std::min(m_base + rb * 8 + r8, M - 1) * K + g * kGroup, 128, n_qx);
                    for (ll u = 0; u < kUnits; ++u) {
                        const ll nf = std::min(nf_base + u, nf_total - 1);
                        chk("codes", nf * G * 1024 + g * 1024, 1024, n_codes);
                        if (mode == 0) chk("meta", g * nf_total * 32 + nf * 32, 32, n_meta);
                    }
                }
            }
            if (S > 1) {
                const ll NJ = 4 * cdiv(MF, WK);
                chk("counter", (tmi * n_tiles + tni) * 4, 4, counters_bytes);
                chk("parts", counters_bytes + ((tmi * n_tiles + tni) * S + sl) * NJ * 512 * 16, NJ * 512 * 16, ws_bytes);
            }
        }
    }
}

// ---- compute-bound kernel -------------------------------------------------------------------------------------------
static void check_mma() {
    int64_t tm, tn;
    compute_bound_tile(M, N, G, mode, tile, split, tm, tn);
    const ll n_tiles = cdiv(N, tn), m_tiles = cdiv(M, tm), S = split, gps = cdiv(G, S), nf_total = N / 16;
    const ll kACopies = tm / 64, kUnits = tn / 16, kWCopies = kUnits / 4, tiles = n_tiles * m_tiles;
    if (cdiv(G, gps) != S) { fail = "mma slices"; return; }
    if (tile == 132 || (tile == 131 && tm == 128)) {           // two per compute unit: a wave's fragments in LDS, places of the three blocks with 192 channels
        std::vector<char> unit(kUnits);
        for (int wave = 0; wave < 4; ++wave) for (int f = 0; f < tn / 64; ++f) {
            const ll u = tn == 256 ? wave * 4 + f : f * 4 + wave;
            chk("LDS weights", (tn == 256 ? wave * 4 : wave) * 1024 + f * (tn == 256 ? 1024 : 4096), 1024, kUnits * 1024);
            chk("LDS metadata", u / kWCopies * 256 + u % kWCopies * 32, 32, 1024);
            if (!fail && unit[u]++) { fail = "a unit twice"; return; }
        }
    }
    for (ll t = 0; t < tiles; ++t) for (ll sl = 0; sl < S; ++sl) {
        const ll tmi = t / n_tiles, tni = t % n_tiles, m_base = tmi * tm, n_base = tni * tn, nf_base = tni * kUnits;
        const ll g_first = sl * gps, Gs = std::min(G - g_first, gps), g_last = g_first + Gs - 1;
        if (Gs < 1) { fail = "mma empty slice"; return; }
        for (ll g = g_first; g <= g_last; ++g) for (int wave = 0; wave < 4; ++wave) {
            for (int hf = 0; hf < 2; ++hf) for (ll c = 0; c < kACopies; ++c) for (int r = 0; r < 8; ++r)
                chk("qx", std::min(m_base + ((wave * 2 + hf) * kACopies + c) * 8 + r, M - 1) * K + g * kGroup, 128, n_qx);
            for (ll u = 0; u < kWCopies; ++u)
                chk("codes", std::min(nf_base + wave * kWCopies + u, nf_total - 1) * G * 1024 + g * 1024, 1024, n_codes);
            if (mode == 0) for (int lane = 0; lane < 64; ++lane) {
                const ll ml = std::min<ll>(lane, kWCopies * 8 - 1);
                chk("meta", g * nf_total * 32 + std::min(nf_base + wave * kWCopies + (ml >> 3), nf_total - 1) * 32 + (ml & 7) * 4, 4, n_meta);
            }
        }
        for (int d = 0; d < 256; ++d) {                        // epilogue constants: 256 of each, clamped
            if (d < 128) chk("sx", m_base * 2 + std::min<ll>(d, (M - m_base - 1) >> 1) * 4, 4, n_sx);
            if (d < 128) chk("scales", n_base * 2 + std::min<ll>(d, ((N - n_base) >> 1) - 1) * 4, 4, n_scales);
            if (mode == 1) chk("rowsum", (m_base + std::min<ll>(d, M - m_base - 1)) * 4, 4, n_rs);
            if (mode == 1 && d < 64) chk("zeros", n_base + std::min<ll>(d, ((N - n_base) >> 2) - 1) * 4, 4, n_zeros);
        }
        if (S > 1) {
            chk("counter", t * 4, 4, counters_bytes);
            chk("parts", counters_bytes + (t * S + sl) * tm * tn * 4, tm * tn * 4, ws_bytes);
        }
    }
}

int main(int argc, char** argv) {
    FILE* f = fopen(argv[1], "r");
    long checked = 0;
    int forced;
    while (fscanf(f, "%lld %lld %lld %d %d %d %lld %d", &M, &N, &K, &mode, &tile, &split, &ws_bytes, &forced) == 8) {
        G = K / kGroup;
        n_codes = N * K / 2; n_meta = mode == 0 ? N * G * 2 : 0; n_scales = 2 * N; n_zeros = mode == 1 ? N : 0;
        n_qx = M * K; n_sx = (2 * M + 3) / 4 * 4; n_rs = 4 * M;       // (token scales are read in whole 4-byte words)
        fail = nullptr;
        parts_end = 0;
        const int wide = M <= 48 * cdiv(M, 64) ? 3 : 4;        // as many tiles of 48 tokens hold them all
        if (tile == 0) check_linear();
        else if (tile == 64) check_stream(wide, true);
        else if (tile == 32 || tile == 16) check_stream(tile / 16, false);
        else if (tile == 65) check_lockstep(2, wide);
        else if (tile == 66) check_lockstep(4, wide);
        else if (tile == 67) check_lockstep(2, 2);
        else if (tile == 68) check_lockstep(2, 1);
        else if (tile >= 69 && tile <= 71) check_astat(tile == 71 ? 64 : tile == 70 ? 32 : 16);
        else if (tile == 130) check_mma8();
        else check_mma();
        // the size of one plan, and not the larger of two: what it touches and no more
        if (!fail && forced && tile >= 128 && parts_end != ws_bytes) { fail = "workspace"; fail_off = 0; fail_len = parts_end; fail_size = ws_bytes; }
        if (fail) {
            printf("M=%lld N=%lld K=%lld mode=%d tile=%d split=%d: %s access [%lld, +%lld) outside %lld bytes\n", M, N, K, mode, tile,
                   split, fail, fail_off, fail_len, fail_size);
            return 1;
        }
        ++checked;
    }
    printf("ok %ld launch plans\n", checked);
    return 0;
}
'''


def _plans(api):
    shapes = [(N, K) for N in (64, 192, 256, 4096, 12288, 22016, 57344) for K in (128, 1152, 4096, 11008, 28672)]
    Ms = (1, 7, 9, 16, 17, 32, 33, 48, 63, 64, 65, 96, 100, 128, 130, 200, 256, 300, 512, 1000, 1024, 4096)
    forced = [(0, 0), (16, 0), (16, 7), (32, 0), (32, 9), (64, 0), (64, 5), (65, 0), (65, 3), (66, 0), (66, 2), (67, 0), (68, 2),
              (69, 0), (69, 5), (70, 0), (71, 0), (71, 3), (128, 0), (128, 3), (129, 0), (129, 2), (130, 0), (130, 2), (130, 5), (131, 0), (131, 2),
              (132, 0)]
    lines = []
    for cfg in forced:
        api.set_gemm_config(*cfg)
        try:
            for N, K in shapes:
                if cfg != (0, 0) and (N, K) not in ((192, 1152), (256, 128), (4096, 4096), (4096, 11008), (22016, 4096), (12288, 1152)):
                    continue                                   # forced configurations: a smaller set of shapes
                for M in Ms:
                    if cfg != (0, 0) and M not in (1, 9, 17, 48, 64, 96, 100, 300, 1024):
                        continue
                    for mode in (0, 1):
                        tile, split = api.query_gemm_config(M, N, K, mode)
                        ws = api.gemm_workspace_bytes(M, N, K, mode)
                        lines.append((M, N, K, mode, tile, split, ws, int(cfg != (0, 0))))
            # more blocks, fragments or tiles than there are counters
            for M, N, K in {(0, 0): [(408, 623680, 128), (139, 3066752, 256)], (64, 5): [(4096, 65664, 256)], (16, 7): [(640, 131072, 256)],
                            (69, 5): [(6000, 4096, 16384)], (71, 3): [(9000, 8192, 5120)], (129, 2): [(33000, 65536, 256)]}.get(cfg, ()):
                lines.append((M, N, K, 1, *api.query_gemm_config(M, N, K, 1), api.gemm_workspace_bytes(M, N, K, 1), int(cfg != (0, 0))))
        finally:
            api.set_gemm_config(0, 0)
    for M in range(1, 17):                                     # one launch: tile code 0 of the checker
        rows = 1 << (M - 1).bit_length()
        for K in (128, 256, 1152, 8192 // rows, 16384 // rows, 32768 // rows):
            lines += [(M, N, K, mode, 0, 0, 0, 0) for N in (64, 320, 5120) for mode in (0, 1) if rows * K <= 32768 and K <= 8192 and K % 128 == 0]
    return lines


def test_every_launch_plan_stays_inside_its_buffers(tmp_path):
    import ctypes

    from paper_2405_04532_amd import api
    L = api.lib()
    plans = _plans(api)
    assert len(plans) > 1500
    src = tmp_path / "bounds.cpp"
    src.write_text(CHECKER)
    exe = tmp_path / "bounds"
    subprocess.check_call(["g++", "-std=c++17", "-O2", "-I", os.path.join(ROOT, "paper_2405_04532_amd", "csrc"), str(src), "-o", str(exe)])
    listing = tmp_path / "plans.txt"
    with open(listing, "w") as f:
        for plan in plans:
            f.write("%d %d %d %d %d %d %d %d\n" % plan)
    out = subprocess.run([str(exe), str(listing)], capture_output=True, text=True)
    assert out.returncode == 0 and out.stdout.startswith("ok"), out.stdout[-2000:]
    assert int(out.stdout.split()[1]) == len(plans)


@pytest.mark.parametrize("right,wrong,plan", [
    # a run that is allowed to reach group G (one past the last) of the last token row: nine groups, the last iteration has one unit
    ("const ll gsel = std::min<ll>(o.g + (e < o.n ? e : 0), G - 1);", "const ll gsel = o.g + e;", "64 256 1152 0 64 4 0 0"),
    # eight waves: a stage of two groups whose second lies past the slice; a token row past M
    ("const ll g = std::min(g_first + st * SG + sg, g_last);", "const ll g = g_first + st * SG + sg;", "100 320 1152 0 130 1 0 1"),
    ("chk(\"qx\", std::min(m_base + rb * 8 + r8, M - 1)", "chk(\"qx\", (m_base + rb * 8 + r8)", "100 320 1152 0 130 1 0 1"),
    # their counters and sums in a workspace of another size
    ("parts_end != ws_bytes", "parts_end != ws_bytes + 256", "96 128 640 0 130 2 393216 1"),
    # sixteen waves: the last waves' groups past the end of the row
    ("const ll col = std::min((g_lo + w * jeff + jp * JP) * kGroup + ((pos ^ (row_local & 15)) * 16), K - 16);",
     "const ll col = (g_lo + w * jeff + jp * JP) * kGroup + ((pos ^ (row_local & 15)) * 16);", "16 64 12416 0 69 4 0 1"),
    # 48 tokens: the second pass read in full
    ("if (rows == 16 && rp * RP + i * 8 / JP >= MF * 16) continue;", "if (rp * RP + i * 8 / JP >= 32) continue;", "48 64 2048 0 71 4 0 1"),
    # tokens of one launch: a row that takes more chunks than its threads hold
    ("rows * K <= 2 * 8 * 512 ? 2 : 8", "2", "16 64 2048 0 0 0 0 0"),
    # a window that ends with the fragments that are multiplied, not with those ahead of them
    ("const ll window = std::min(nfr - fi0, 2 * R) * G * 1024;", "const ll window = std::min(nfr - fi0, R) * G * 1024;", "16 24576 4096 0 69 256 0 1"),
    # 192 channels: units of the wide tile
    ("const ll u = tn == 256 ? wave * 4 + f : f * 4 + wave;", "const ll u = wave * 4 + f;", "300 832 1152 1 131 1 0 1")])
def test_the_checker_catches_a_planted_overrun(tmp_path, right, wrong, plan):
    """Mistakes planted in the host model, the first of which once faulted on the GPU, must be reported."""
    assert CHECKER.count(right) == 1
    listing = tmp_path / "plans.txt"
    listing.write_text(plan + "\n")
    for source, status in ((CHECKER, 0), (CHECKER.replace(right, wrong), 1)):
        src, exe = tmp_path / "bounds.cpp", tmp_path / "bounds"
        src.write_text(source)
        subprocess.check_call(["g++", "-std=c++17", "-O2", "-I", os.path.join(ROOT, "paper_2405_04532_amd", "csrc"), str(src), "-o", str(exe)])
        out = subprocess.run([str(exe), str(listing)], capture_output=True, text=True)
        assert out.returncode == status and ("outside" in out.stdout or "left out" in out.stdout or "window" in out.stdout) == bool(status), out.stdout


@pytest.mark.parametrize("M,N,K,mode,tile,nwg", [(130, 12288, 4096, 0, 71, 80), (65, 10240, 8192, 0, 70, 80), (100, 10240, 8192, 1, 70, 64),
                                                 (300, 8192, 8192, 1, 70, 24), (700, 22016, 4096, 0, 132, 1),
                                                 (130, 4096, 3968, 0, 70, 48), (65, 6144, 3968, 0, 70, 80), (130, 6144, 3584, 0, 70, 48)])
def test_side_by_side_tiles_share_an_xcd(M, N, K, mode, tile, nwg):
    """Activation-stationary tiles side by side get a multiple of eight workgroups each (the same XCD for a fragment run in
    every token tile) and hold all of K, whatever K is; a small remainder behind a full round stays with the two-per-CU tile."""
    from paper_2405_04532_amd import api
    assert api.query_gemm_config(M, N, K, mode) == (tile, nwg)


@pytest.mark.parametrize("M,N,K,mode,tile", [(80, 4096, 11008, 0, 64), (88, 4480, 11008, 0, 64), (96, 5120, 11008, 0, 32), (80, 4096, 11008, 1, 64),
                                             (80, 4608, 11008, 1, 32), (65, 5120, 11008, 1, 32)])
def test_tiles_of_48_tokens_in_place_of_32(M, N, K, mode, tile):
    """Long rows: up to a width where the 32-token tiles, a block per workgroup, are as fast."""
    from paper_2405_04532_amd import api
    assert api.query_gemm_config(M, N, K, mode)[0] == tile


@pytest.mark.parametrize("M,N,K,mode,tile", [(130, 16384, 4096, 1, 71), (144, 15872, 3584, 1, 71), (130, 16384, 2560, 0, 66), (65, 14336, 3072, 0, 71),
                                             (130, 15872, 4096, 0, 130), (112, 13376, 7808, 0, 130)])
def test_short_rows_are_not_cut(M, N, K, mode, tile):
    """One token tile: the eight-wave kernel takes k-slices of short rows only where they are ahead of tiles that exchange nothing."""
    from paper_2405_04532_amd import api
    assert api.query_gemm_config(M, N, K, mode)[0] == tile


def test_workspaces_hold_what_their_kernels_exchange():
    """110 tokens x 5120 x 12288: two k-slices of 96 tiles of 112 tokens x 128 channels, of which each of four waves hands over two
    fragments of every 64 channels; one token of 11008: one workgroup holds all of K, and nothing is exchanged."""
    from paper_2405_04532_amd import api
    assert api.query_gemm_config(110, 12288, 5120) == (130, 2)
    assert api.gemm_workspace_bytes(110, 12288, 5120) == (256 << 10) + 2 * 96 * (4 * 2 * 512 * 16)
    for mode in (0, 1):
        assert api.query_gemm_config(1, 4096, 11008, mode)[0] == 69 and api.gemm_workspace_bytes(1, 4096, 11008, mode) == 0


@pytest.mark.parametrize("B,H,Hkv,S,ranges", [(1, 32, 32, 640, 1), (1, 32, 32, 1023, 1), (1, 32, 32, 1024, 2), (1, 32, 32, 8192, 8), (4, 32, 8, 768, 1),
                                              (1, 32, 8, 8192, 8), (12, 32, 8, 4096, 2), (16, 32, 8, 8192, 2), (17, 32, 8, 8192, 1), (24, 32, 8, 8192, 1),
                                              (31, 32, 8, 8192, 1)])
def test_ranges_of_a_sequence(B, H, Hkv, S, ranges):
    """The host knows how long a sequence may become and not how long it is: caches are cut, which takes a second launch, where that
    costs short sequences little (192 pairs of 128 tokens in caches for 4096 took 9.0 us in four ranges and 3.9 whole)."""
    from paper_2405_04532_amd import api
    assert api.kv4_attention_workspace_bytes(B, H, Hkv, S) == (B * H * 130 * 4 * ranges if ranges > 1 else 0)


TILES = r'''
#include "qoq_tiles.h"
#include <cstdio>
int main()
{
    long long M, N, K, S, tm, tn;
    int mode, tile;
    while (scanf("%lld %lld %lld %d %d %lld", &M, &N, &K, &mode, &tile, &S) == 6) {
        int64_t a, b;
        qoq::compute_bound_tile(M, N, K / qoq::kGroup, mode, tile, S, a, b);
        printf("%lld %lld\n", (long long)a, (long long)b);
    }
}
'''


@pytest.fixture(scope="module")
def tiles_of(tmp_path_factory):
    """Tokens and channels of the tiles that plans of the compute-bound kernels run, from the header that the library includes."""
    d = tmp_path_factory.mktemp("tiles")
    (d / "tiles.cpp").write_text(TILES)
    subprocess.check_call(["g++", "-std=c++17", "-O1", "-I", os.path.join(ROOT, "paper_2405_04532_amd", "csrc"), str(d / "tiles.cpp"), "-o", str(d / "tiles")])

    def ask(plans):
        out = subprocess.run([str(d / "tiles")], input="\n".join("%d %d %d %d %d %d" % p for p in plans), capture_output=True, text=True, check=True).stdout
        return [tuple(map(int, line.split())) for line in out.splitlines()]
    return ask


def test_group_mode_keeps_the_tall_narrow_tile(tiles_of):
    """256 x 192 in group mode, whatever the shape: two of 128 x 192 per compute unit took 0.95 of the speed; per channel they are ahead."""
    shapes = [(951, 12224, 256), (393, 23936, 256), (2221, 5248, 256), (1500, 12288, 4096), (2971, 3776, 1280), (326, 23360, 2688)]
    assert set(tiles_of([(*s, 0, 131, 1) for s in shapes])) == {(256, 192)}
    assert set(tiles_of([(*s, 1, 131, 1) for s in shapes])) == {(128, 192)}
    assert set(tiles_of([(*s, m, 131, 2) for s in shapes for m in (0, 1)])) == {(256, 192)}


@pytest.mark.parametrize("M,N,K,tile", [(1920, 3648, 384, 129), (2735, 2240, 512, 129), (852, 9152, 640, 129), (227, 21888, 3456, 129), (256, 18752, 4736, 129),
                                        (370, 15808, 5120, 129), (1657, 2816, 512, 131), (945, 5952, 640, 131), (478, 11904, 2816, 131), (1992, 21248, 896, 131)])
def test_narrow_tiles_only_where_they_are_ahead(M, N, K, tile):
    """Per channel, in place of 128 x 256 and 256 x 256 tiles: not where the compute units' second workgroup comes on top of short rows, nor
    where few token tiles wait for many weights."""
    from paper_2405_04532_amd import api
    assert api.query_gemm_config(M, N, K, 1) == (tile, 1)


def test_two_per_compute_unit_keep_256_channels_for_short_rows(tiles_of):
    wide = [(1586, 11200, 768, 0), (3464, 5184, 640, 0), (763, 24384, 1024, 0), (2562, 4544, 1152, 0), (623, 19520, 256, 1), (861, 12416, 256, 1), (1063, 10688, 512, 1)]
    narrow = [(548, 16832, 7168, 0), (1382, 8576, 1280, 0), (328, 27584, 13696, 1), (300, 25600, 640, 1),
              (129, 320, 5120, 0), (300, 832, 5120, 0), (257, 448, 5248, 0), (129, 320, 5120, 1)]
    assert tiles_of([(*s, 132, 1) for s in wide + narrow]) == [(128, 256)] * len(wide) + [(128, 192)] * len(narrow)
