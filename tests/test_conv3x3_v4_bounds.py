"""Host-side emulation of the index arithmetic of the persistent 3x3 convolution kernel
(conv3x3_v4_body in csrc/dnb_conv_f32_fast.hip, as k_conv3x3_v4 and as the backward chain's
k_dgrad3_v4): for every workgroup, tile, thread and staging slot it recomputes the addresses the kernel
forms -- global loads of the input rows, packed-weight loads (fragment order, held against the order the
packing kernel writes), LDS stores of the staged rows, LDS operand reads of the nine taps, the statistics
scratch and the output stores; in the backward form also the feature loads, the stores of the corrected
slice (every element once) and the partial sums (every slot once, zeros from workgroups without a tile)
-- with the kernel's own constants (plane pitch 144, row pitch W + 4, 512 workgroups
dealt to 8 XCDs) and checks that each stays inside its buffer and that every tile is taken exactly
once.  An earlier version of the kernel overran the last staged row by one float; this is the
check that found it.  CPU only: nothing is launched."""
import pytest


def wfrag(K16, mtile, chunk, lane):  # offset of a lane's four weights inside one tap's block
    return (mtile*(K16>>4)+chunk)*256+lane*4


def wunfrag(e, K16):  # position inside one tap's block -> row, channel, as the packing kernel writes it
    mt=e//(16*K16); r=e-mt*16*K16; lane=(r>>2)&63
    return mt*16+(lane&15), (r>>8)*16+4*(r&3)+(lane>>4)


def check(n, cin, cout, H, W, label, sample=None, bwd=False):
    HW=H*W; mtiles=(cout+15)//16; M16=mtiles*16; K16=(cin+15)//16*16; nch=K16//16
    assert (mtiles,nch) in ((1,3),(3,1)) and W in (8,16,32) and HW%64==0
    MT,NCH=mtiles,nch; ROWS=NCH*16; RW=W+4; TR=64//W; NR=TR+2; W4=W//4; CS=144
    assert NR*RW<=CS
    PER=NR*W4; TOTAL=ROWS*PER; U=(TOTAL+255)//256; BUF=ROWS*CS+4; SST0=2*BUF
    assert not bwd or (MT,NCH)==(3,1)  # (what k_dgrad3_v4 is instantiated for)
    lds_floats=2*(NCH*16*144+4)+(0 if bwd else 2*4*mtiles*16*3)
    static_bytes=(3*128*4+MT*16*16+4*MT*16*8) if bwd else 0  # coefficients, BN2's constants, its sums
    gl_written={}; part2={}
    tpi=HW//64; total_tiles=tpi*n
    G=(total_tiles+7)//8*8 if total_tiles<512 else 512
    tpx=(total_tiles+7)>>3; wgx=G>>3
    in_elems=n*cin*HW; out_elems=n*cout*HW; w_elems=9*M16*K16
    wgs=range(G) if sample is None or G<=2*sample else list(range(sample))+list(range(G-sample,G))
    full=len(list(wgs))==G; done=set(); bad=0
    for b in wgs:
        xcd=b&7; slot=b>>3; t_lo=xcd*tpx; t_hi=min(total_tiles,t_lo+tpx); tile=t_lo+slot
        it=0
        if bwd:  # the workgroup's partial of every output channel, or zeros if it has no tile
            for m in range(cout): part2[m*G+b]=part2.get(m*G+b,0)+1
        while tile<t_hi:
            assert tile not in done; done.add(tile)
            img=tile//tpi; y0=(tile-img*tpi)*TR
            for tid in range(256):
                lane=tid&63; wave=tid>>6; j=lane&15; g=lane>>4
                for u in range(U):
                    idx=min(u*256+tid,TOTAL-1); sch=idx//PER; rem=idx-sch*PER; sry=rem//W4; sgo=4*(rem-sry*W4)
                    slo=sch*CS+sry*RW+4+sgo
                    y=min(max(y0-1+sry,0),H-1)
                    a=img*cin*HW+min(sch,cin-1)*HW+y*W+sgo
                    if not(0<=a and a+3<in_elems): bad+=1
                    if u*256+tid<TOTAL:
                        for boff in (0,BUF):
                            if not(0<=boff+slo and boff+slo+3<boff+BUF-4): bad+=1
                    if bwd and sch<cin and 1<=sry<=TR and u*256+tid<TOTAL:
                        gq=(img*cin+sch)*HW+(y0-1+sry)*W+sgo  # gl [n][cin][HW], four pixels
                        if not(0<=gq and gq+3<in_elems): bad+=1
                        gl_written[gq]=gl_written.get(gq,0)+1
                for t in range(9):
                    for a_ in range(MT):
                        for ci in range(NCH):
                            wa=t*M16*K16+wfrag(K16,a_,ci,lane)
                            if not(0<=wa and wa+3<w_elems): bad+=1
                            for ks in range(4):  # the channel whose plane the ks-th product reads
                                if wunfrag(wa-t*M16*K16+ks,K16)!=(a_*16+j,ci*16+4*ks+g): bad+=1
                p=16*wave+j; base=g*CS+(p//W+1)*RW+4+(p%W)
                for boff in (0,BUF):
                    for ci in range(NCH):
                        for di in (-1,0,1):
                            for dj in (-1,0,1):
                                for ks in range(4):
                                    l=boff+base+(ci*16+4*ks)*CS+di*RW+dj
                                    if not(boff<=l<boff+BUF): bad+=1
                q=(tile-img*tpi)*64+p
                assert q<HW
                for a_ in range(MT):
                    for r in range(4):
                        m=a_*16+4*g+r
                        if m<cout:
                            o=img*cout*HW+q+m*HW
                            if not(0<=o<out_elems): bad+=1
                        if bwd: continue
                        sidx=SST0+(((1*4+wave)*(MT*16))+a_*16+4*g+r)*3
                        if not(sidx+2<lds_floats): bad+=1
            tile+=wgx; it+=1
    assert (not full) or done==set(range(total_tiles)), label
    if bwd:
        assert all(v==1 for v in gl_written.values()) and all(v==1 for v in part2.values()), label
        if full:
            assert sorted(gl_written)==list(range(0,n*cin*HW,4)), label
            assert sorted(part2)==list(range(cout*G)), label
    return bad, lds_floats * 4 + static_bytes


CASES = [
    (2, 48, 12, 8, 8, "fwd 8x8", None),
    (2, 12, 48, 8, 8, "dgrad 8x8", None),
    (2, 48, 12, 32, 32, "fwd 32x32", None),
    (3, 12, 48, 16, 16, "dgrad 16x16 n3", None),
    (64, 48, 12, 32, 32, "fwd, first block of DenseNet-BC-100 at batch 64", 6),
    (64, 12, 48, 32, 32, "dgrad, first block", 6),
    (64, 48, 12, 16, 16, "fwd, second block", 6),
    (64, 12, 48, 16, 16, "dgrad, second block", 6),
    (64, 48, 12, 8, 8, "fwd, third block", None),
    (64, 12, 48, 8, 8, "dgrad, third block", None),
    (4, 40, 12, 8, 8, "fwd, 40 input channels (channel tail)", None),
    (2, 12, 40, 8, 16, "dgrad, 40 output channels, 8x16 image", None),
]


BWD_CASES = [
    (2, 12, 48, 8, 8, "8x8, workgroups without a tile", None),
    (3, 16, 33, 16, 16, "16x16, 16 and 33 channels", None),
    (2, 8, 40, 8, 16, "8x16, 8 and 40 channels", None),
    (1, 12, 48, 32, 32, "32x32", None),
    (64, 12, 48, 32, 32, "first block of DenseNet-BC-100 at batch 64", 6),
    (70, 12, 48, 16, 16, "16x16 at batch 70", 6),
]


@pytest.mark.parametrize("n,cin,cout,H,W,label,sample", BWD_CASES, ids=[c[5] for c in BWD_CASES])
def test_every_access_of_the_backward_form_is_in_bounds(n, cin, cout, H, W, label, sample):
    bad, lds_bytes = check(n, cin, cout, H, W, label, sample, bwd=True)
    assert bad == 0
    assert lds_bytes <= 64 * 1024


@pytest.mark.parametrize("n,cin,cout,H,W,label,sample", CASES, ids=[c[5] for c in CASES])
def test_every_access_of_the_persistent_3x3_kernel_is_in_bounds(n, cin, cout, H, W, label, sample):
    bad, lds_bytes = check(n, cin, cout, H, W, label, sample)
    assert bad == 0
    assert lds_bytes <= 64 * 1024


def check_wave_per_m_tile(n, cin, cout, H, W):
    """k_dgrad3_wpm: NW waves of one M-tile each over the 64 pixels of a tile, 4*NK staged channels."""
    HW=H*W; M16=(cout+15)//16*16; K16=(cin+15)//16*16; NW=6 if M16<=96 else 8; NK=6 if cin<=24 else 8
    assert 64<cout<=128 and 16<cin<=32 and W in (8,16,32) and HW%64==0
    NT=NW*64; ROWS=4*NK; RW=W+4; TR=64//W; NR=TR+2; W4=W//4; CS=144; PER=NR*W4; TOTAL=ROWS*PER; U=(TOTAL+NT-1)//NT
    BUF=ROWS*CS+4; assert NR*RW<=CS and 2*BUF%4==0
    tpi=HW//64; total=tpi*n; G=(total+7)//8*8 if total<512 else 512; tpx=(total+7)>>3
    staged={}; written={}; gl={}; part={}; done=set()
    for b in range(G):
        tile=(b&7)*tpx+(b>>3); t_hi=min(total,(b&7)*tpx+tpx)
        if tile>=t_hi:
            for m in range(min(cout,NT)): part[m*G+b]=part.get(m*G+b,0)+1
            continue
        for wave in range(NW):
            for lane in range(64):
                for r in range(4):
                    m=wave*16+4*(lane>>4)+r
                    if lane&15==0 and m<cout: part[m*G+b]=part.get(m*G+b,0)+1
        while tile<t_hi:
            assert tile not in done; done.add(tile)
            img=tile//tpi; y0=(tile-img*tpi)*TR; first=b==0 and len(done)==1
            for tid in range(NT):
                for u in range(U):
                    idx=min(u*NT+tid,TOTAL-1); sch=idx//PER; rem=idx-sch*PER; sry=rem//W4; sgo=4*(rem-sry*W4)
                    slo=sch*CS+sry*RW+4+sgo
                    assert 0<=slo and slo+3<BUF-4 and slo%4==0
                    o=min(sch,cin-1)*HW+min(max(y0-1+sry,0),H-1)*W+sgo
                    assert 0<=o and o+3<cin*HW
                    if u*NT+tid<TOTAL:
                        if first:
                            for e in range(4): staged[slo+e]=(sch,sry-1,sgo+e)
                        if sch<cin and 1<=sry<=TR:
                            q=(img*cin+sch)*HW+(y0-1+sry)*W+sgo
                            gl[q]=gl.get(q,0)+1
            for wave in range(NW):
                mt=min(wave,(M16>>4)-1)
                for lane in range(64):
                    j=lane&15; g=lane>>4; base=g*CS+(j//W+1)*RW+4+j%W
                    if first:
                        for t9 in range(9):
                            for kk in range(NK):
                                wa=wfrag(K16,mt,kk//4,lane)+kk%4
                                assert wa<M16*K16 and wunfrag(wa,K16)==(mt*16+j,4*kk+g)
                                for t in range(4):
                                    l=base+4*kk*CS+(t9//3-1+16*t//W)*RW+t9%3-1+16*t%W
                                    assert 0<=l<BUF
                                    p=16*t+j; y=p//W+t9//3-1; x=p%W+t9%3-1  # the tap's row and column
                                    assert staged.get(l)==((4*kk+g,y,x) if 0<=x<W else None)
                    for r in range(4):
                        m=wave*16+4*g+r
                        assert min(m,cout-1)*HW+(tile-img*tpi)*64+48+j<cout*HW
                        if m<cout:
                            for t in range(4):
                                o=(img*cout+m)*HW+(tile-img*tpi)*64+16*t+j
                                written[o]=written.get(o,0)+1
            tile+=G>>3
    assert done==set(range(total))
    assert len(written)==n*cout*HW and all(v==1 for v in written.values())
    assert sorted(gl)==list(range(0,n*cin*HW,4)) and all(v==1 for v in gl.values())
    assert sorted(part)==list(range(cout*G)) and all(v==1 for v in part.values())
    return 2*BUF*4+3*128*4+NW*16*16


@pytest.mark.parametrize("n,cin,cout,H,W", [(1, 24, 96, 32, 32), (3, 24, 96, 8, 8), (5, 17, 65, 8, 16), (1, 32, 128, 4, 16),
                                            (2, 25, 100, 16, 8), (1, 20, 81, 2, 32), (36, 24, 72, 32, 32),
                                            # the other pairs of waves and K-steps: eight and six, six and eight
                                            (1, 32, 128, 2, 32), (1, 24, 112, 2, 32), (2, 24, 112, 4, 16), (2, 17, 113, 8, 8),
                                            (1, 30, 90, 2, 32), (2, 32, 96, 4, 16), (2, 28, 80, 8, 8)])
def test_every_access_of_the_wave_per_m_tile_form_is_in_bounds(n, cin, cout, H, W):
    assert check_wave_per_m_tile(n, cin, cout, H, W) <= 80 * 1024  # two workgroups a CU
