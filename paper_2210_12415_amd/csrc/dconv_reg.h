// Registration of one direct-convolution tile configuration with the kernel table.
#pragma once
#include "dslab.h"
#include "dstream.h"

// BM x BN output tile, WGM x WGN waves, NS weight stages
#define ALT_DCONV(BM, BN, WGM, WGN, NS)                                                                          \
    const bool reg_dconv_##BM##x##BN##_w##WGM##x##WGN##_s##NS =                                                  \
        (igemm_register(IgemmLaunch{"bf16_" #BM "x" #BN "x64_direct_w" #WGM "x" #WGN "_s" #NS, ALT_BF16, BM, BN,  \
                                    64, LOAD_VEC, LOAD_VEC, NS - 1, 1, 0, nullptr,                               \
                                    &dconv_launch<BM, BN, WGM, WGN, 1, NS, 64>, WGM, WGN, 1}),                   \
         true)

// the same with KW K groups of WGM x WGN waves each and K steps of BK channels
#define ALT_DCONV_KW(BM, BN, WGM, WGN, KW, NS, BK)                                                               \
    const bool reg_dconv_##BM##x##BN##_w##WGM##x##WGN##x##KW##_s##NS##_b##BK =                                   \
        (igemm_register(IgemmLaunch{"bf16_" #BM "x" #BN "x" #BK "_direct_w" #WGM "x" #WGN "x" #KW "_s" #NS,       \
                                    ALT_BF16, BM, BN, BK, LOAD_VEC, LOAD_VEC, NS - 1, 1, 0, nullptr,             \
                                    &dconv_launch<BM, BN, WGM, WGN, KW, NS, BK>, WGM, WGN, KW}),                 \
         true)

// streaming kernel (dstream.h): BM x BN tile, KW K groups of WGM x WGN waves, NS stages of BK channels
#define ALT_DSTREAM(BM, BN, WGM, WGN, KW, NS, BK)                                                                \
    const bool reg_dstream_##BM##x##BN##x##BK##_w##WGM##x##WGN##x##KW##_s##NS =                                  \
        (igemm_register(IgemmLaunch{"bf16_" #BM "x" #BN "x" #BK "_stream_w" #WGM "x" #WGN "x" #KW "_s" #NS,       \
                                    ALT_BF16, BM, BN, BK, LOAD_VEC, LOAD_VEC, NS - 1, 1, 0, nullptr,             \
                                    &dstream_launch<BM, BN, WGM, WGN, KW, NS, BK>, WGM, WGN, KW, 1}),            \
         true)

// channel-planar kernel (dplanar.h): BM x BN tile, KW K groups of WGM x WGN waves; named rplanar for channels that are no multiple
// of 64 or more than LDS holds at once
#define ALT_DPLANAR_(BM, BN, WGM, WGN, KW, RAGGED, MNAME)                                                        \
    const bool reg_d##MNAME##_##BM##x##BN##_w##WGM##x##WGN##x##KW =                                              \
        (igemm_register(IgemmLaunch{"bf16_" #BM "x" #BN "x64_" #MNAME "_w" #WGM "x" #WGN "x" #KW, ALT_BF16, BM, BN, \
                                    64, LOAD_VEC, LOAD_VEC, 0, 0, 0, nullptr,                                    \
                                    &dplanar_launch<BM, BN, WGM, WGN, KW>, WGM, WGN, KW, 2, 0, 0, RAGGED}),      \
         true)
#define ALT_DPLANAR(BM, BN, WGM, WGN, KW) ALT_DPLANAR_(BM, BN, WGM, WGN, KW, 0, planar); ALT_DPLANAR_(BM, BN, WGM, WGN, KW, 1, rplanar)

// the streaming kernel for B stored [K][N] (row-major): the same tiles, B read through LDS transpose reads
#define ALT_DSTREAM_KN(BM, BN, WGM, WGN, KW, NS, BK)                                                             \
    const bool reg_dstream_kn_##BM##x##BN##x##BK##_w##WGM##x##WGN##x##KW##_s##NS =                               \
        (igemm_register(IgemmLaunch{"bf16_" #BM "x" #BN "x" #BK "_streamkn_w" #WGM "x" #WGN "x" #KW "_s" #NS,     \
                                    ALT_BF16, BM, BN, BK, LOAD_VEC, LOAD_VEC, NS - 1, 1, 0, nullptr,             \
                                    &dstream_launch<BM, BN, WGM, WGN, KW, NS, BK, true>, WGM, WGN, KW, 1, 1}),   \
         true)

// the streaming kernel over filter taps: MODE kTapsUniform (named taps) or kTapsRagged (named rtaps), T and TNAME the element type
#define ALT_DTAPS_(T, TNAME, DT, BM, BN, WGM, WGN, KW, NS, BK, MODE, MNAME)                                      \
    const bool reg_dtaps_##TNAME##_##BM##x##BN##x##BK##_w##WGM##x##WGN##x##KW##_s##NS##_##MNAME =                \
        (igemm_register(IgemmLaunch{#TNAME "_" #BM "x" #BN "x" #BK "_" #MNAME "_w" #WGM "x" #WGN "x" #KW "_s" #NS, \
                                    DT, BM, BN, BK, LOAD_VEC, LOAD_VEC, NS - 1, 1, 0, nullptr,                   \
                                    &dstream_launch<BM, BN, WGM, WGN, KW, NS, BK, false, MODE, T>, WGM, WGN, KW, 1, 0, MODE}), \
         true)
#define ALT_DTAPS(BM, BN, WGM, WGN, KW, NS, BK) ALT_DTAPS_(bf16_tag, bf16, ALT_BF16, BM, BN, WGM, WGN, KW, NS, BK, kTapsUniform, taps)
#define ALT_DRTAPS(BM, BN, WGM, WGN, KW, NS, BK) ALT_DTAPS_(bf16_tag, bf16, ALT_BF16, BM, BN, WGM, WGN, KW, NS, BK, kTapsRagged, rtaps)
#define ALT_DRTAPS_F32(BM, BN, WGM, WGN, KW, NS, BK) ALT_DTAPS_(float, f32, ALT_F32, BM, BN, WGM, WGN, KW, NS, BK, kTapsRagged, rtaps)
// ragged K with B stored [K][N]
#define ALT_DRSTREAM_KN(BM, BN, WGM, WGN, KW, NS, BK)                                                            \
    const bool reg_drstream_kn_##BM##x##BN##x##BK##_w##WGM##x##WGN##x##KW##_s##NS =                              \
        (igemm_register(IgemmLaunch{"bf16_" #BM "x" #BN "x" #BK "_rtapskn_w" #WGM "x" #WGN "x" #KW "_s" #NS,      \
                                    ALT_BF16, BM, BN, BK, LOAD_VEC, LOAD_VEC, NS - 1, 1, 0, nullptr,             \
                                    &dstream_launch<BM, BN, WGM, WGN, KW, NS, BK, true, kTapsRagged>, WGM, WGN, KW, 1, 1, kTapsRagged}), \
         true)

// patch-resident kernel over slabs of BK channels (dslab.h): BM x BN tile, KW K groups of WGM x WGN waves
#define ALT_DSLAB(BM, BN, WGM, WGN, KW, BK)                                                                      \
    const bool reg_dslab_##BM##x##BN##x##BK##_w##WGM##x##WGN##x##KW =                                            \
        (igemm_register(IgemmLaunch{"bf16_" #BM "x" #BN "x" #BK "_slab_w" #WGM "x" #WGN "x" #KW, ALT_BF16, BM, BN, \
                                    BK, LOAD_VEC, LOAD_VEC, 2, 1, 0, nullptr,                                    \
                                    &dslab_launch<BM, BN, WGM, WGN, KW, BK>, WGM, WGN, KW, 4, 0, kTapsRagged}),  \
         true)
