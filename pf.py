import sys,os
sys.path.insert(0,'/root/repo/perf'); sys.path.insert(0,os.getcwd())
import torch,cases
for heads,seqs,lo,hi,pre in [('32/8',1,64,64,0),('32/8',1,256,256,0),('32/8',1,512,512,0),('32/8',1,1000,1000,0),('32/8',1,2000,2000,0),('32/8',1,3000,3000,0),('32/8',1,4000,4000,0),('32/8',1,6000,6000,0),('32/8',3,400,1100,0),('32/8',6,300,3000,2000),('32/4',1,1000,1000,0),('32/4',1,2000,2000,0),('32/4',1,4000,4000,0),('32/4',2,3000,5000,0),('64/8',1,1000,1000,0),('64/8',1,2000,2000,0),('64/8',1,4000,4000,0),('4/2',4,100,900,0),('4/2',1,2000,2000,0),('4/2',1,16000,16000,0),('32/8',1,16000,16000,0),('32/4',1,300,300,4000)]:
    s=cases.prepare({'kind':'pattn','heads':heads,'seqs':seqs,'lo':lo,'hi':hi,'prefix':pre},3)
    row=[];ref=None
    for c in (0,1,2,3,4):
        os.environ['PF']=str(c)
        for _ in range(3): o=cases.run(s)
        torch.cuda.synchronize()
        if ref is None: ref=o.clone()
        d=(o.float()-ref.float()).abs().max().item()
        e0=torch.cuda.Event(enable_timing=True);e1=torch.cuda.Event(enable_timing=True);best=1e9
        for r in range(3):
            e0.record()
            for _ in range(10): cases.run(s)
            e1.record();torch.cuda.synchronize();best=min(best,e0.elapsed_time(e1)*100)
        row.append('c%d %.1f%s'%(c,best,'' if d==0 else ' DIFF %g'%d))
    print(heads,seqs,lo,hi,pre,' '.join(row),flush=True)
    del s
